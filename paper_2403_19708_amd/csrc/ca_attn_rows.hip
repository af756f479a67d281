// Causal attention for plans in which every (conversation, kv head) has few stacked query rows (3 to 32: decode steps of
// grouped-query models, very short turns; Sections 2.1, 3.2.2, 3.4).  Each key and value byte is used for a few rows only,
// so the kernel is bound by HBM: it streams the context once, at the rate of a large copy, and keeps the matrix cores fed
// on the side.
//
//   * Nothing is shared between the wavefronts of a workgroup while they walk: wavefront w takes pages w, w + NWV, ... of
//     the item for ALL its rows, through an LDS ring of its own (a page of K and V per stage, 8 KiB at D = 128), filled by
//     global_load_lds and released by its own s_waitcnt.  No barrier until the end of an item; eight wavefronts of a
//     compute unit keep about 100 KiB in flight, which is what HBM's latency asks for at 6 TB/s.  (The tile kernel of
//     ca_attn_dma.hip walks 32-key tiles in lock step and pads 8 rows to 32: 139 us for 64 conversations of 1024 to 4096
//     tokens, 8 kv heads, 671 to 679 MB, where this kernel takes 118 back to back and 124 with other kernels between.)
//   * S^T = K Q^T with v_mfma_f32_16x16x32_bf16 (16 keys x 16 rows), O^T += V^T P^T with v_mfma_f32_16x16x16_bf16: the C
//     registers of the first, rounded to bf16, are the B operand of the second.  Softmax as in the tile kernel: scale and
//     log2(e) folded into the rotated query, the reference maximum enters as the accumulator and is raised lazily in long runs.
//   * Keys are rotated in registers between the LDS read and the matrix instruction: a lane's operand pieces of one key
//     hold both members of every rotary pair.  (cos, sin) advance by a constant rotation from page to page.
//   * Workgroups of four wavefronts, two to a compute unit (of eight where nothing is cut and units are few).  With enough to
//     stream the pages of all (conversation, kv head) units, laid end to end, are cut into equal runs, one per workgroup: all have the
//     same number of bytes whatever the lengths.
//     With less (one conversation: 11 MB) the time is a chain of dependent steps and a workgroup has one share, whose
//     description brings everything the first loads need.  Clock stamps of that chain (2777 tokens, 8 kv heads, 8 rows, 3 pages a
//     wavefront): description 0.4 us, first loads landed 4.2, walk 7.1, wavefronts merged 7.8, share acknowledged and
//     counted 9.4, shares merged 11.6.  A compute unit takes 16 cycles for a load instruction of 1 KiB and about 45 KB/us from
//     beyond its cache, and a wavefront alone on its SIMD 0.9 us a page, most of it the rotation: hence few loads (each
//     query row is fetched and rotated once per workgroup, and a share is read 16 bytes a lane) and few pages a wavefront.
//     With eight wavefronts of 16 pages a share, each fetching the queries by itself, this took 14.4 us; the
//     decode step of that conversation over 80 layers 1506 -> 1279 us, of 8 of 700 to 1800 tokens over 20 layers 620 -> 469, of 64 of
//     200 to 600 tokens 730 -> 602.
//   * A share that is not a whole unit leaves unnormalised sums, maximum and denominator, and the workgroup that finishes a
//     unit's last share merges them: no second launch (a combine kernel behind a decode step's attention cost 4 us plus the
//     gap in front of it).  Shares are written through to memory; with release fences instead, each of which writes back a
//     die's L2, the kernel took 335 us instead of 121.
#include "ca_internal.h"
#include "ca_device.h"

namespace ca {

namespace {

// f over the four lanes l, l ^ 16, l ^ 32, l ^ 48, which have the keys of one row
template <typename F>
__device__ inline float over_row(float v, F f) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// D, rotary style, NB = 16-row blocks (rows <= 16 NB), NWV = wavefronts of a workgroup, ONE = workgroup w has item w only (else
// the items [wg_first[w], wg_first[w + 1]))
template <int D, int STYLE, int NB, int NWV, bool ONE>
__global__ __launch_bounds__(64 * NWV, 2) void attn_rows_kernel(AttnArgs a) {
    constexpr int HALF = D / 2;
    constexpr int PPR = D / 8;                // 16-byte pieces per row
    constexpr int KPC = 64 / PPR;             // keys per 1 KiB chunk
    constexpr int CPP = kPageSize / KPC;      // chunks of a page per array
    constexpr int CH = 1024 + KPC * 16;       // chunk stride in LDS
    constexpr int PAGE = CPP * CH;            // bytes of one page of K (or V) in LDS
    constexpr int STAGE = 2 * PAGE;
    constexpr int NS = D == 128 ? 2 : 4;      // stages: 16 KiB in flight per wavefront at most
    constexpr int LOADS = 2 * CPP;            // load instructions per page
    constexpr int KK = D / 32;                // k-steps of the score product
    constexpr int DB = D / 16;                // 16-dim blocks of O^T
    constexpr int ROWS = 16 * NB;
    constexpr int OSTR = D + 4;               // row stride of the merge buffer (floats): conflict-free 16-byte accesses
    constexpr int QSTR = 2 * D + 16;          // row stride of the rotated queries (bytes): conflict-free 16-byte accesses
    // How far (exponent units) a score may lie above the reference maximum.  A new maximum that becomes the reference has a
    // probability of exactly 1, and those are a row's largest.  In walks of a few pages it is felt where the reference stays behind:
    // the error against 64 bits over 39 batches of shares and short contexts is 0.95 to 0.99 times that of workgroups of eight
    // wavefronts with a headroom of 8 and 16 pages a share, with a headroom of 8 here 0.95 to 1.035.  It costs up to 2.7 % of a decode
    // step (one conversation of 2777 tokens, 80 layers: 0.1 to 0.6 %).  Long runs keep theirs.
    constexpr float kHeadroom = ONE ? 0.0f : 8.0f;
    constexpr int RING = NWV * NS * STAGE, MERGE = NWV * ROWS * OSTR * 4;
    constexpr int SMEM = RING > MERGE ? RING : MERGE;
    static_assert(SMEM + ROWS * QSTR + NWV * ROWS * 8 + 256 <= (NWV == 4 ? 80 : 160) * 1024, "LDS budget");

    __shared__ __attribute__((aligned(16))) uint8_t smem[SMEM];
    __shared__ __attribute__((aligned(16))) uint8_t q_rot[ROWS * QSTR];
    __shared__ float red_m[NWV][ROWS], red_l[NWV][ROWS];
    __shared__ int32_t is_last;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int q4 = lane >> 4, m16 = lane & 15;
    const int G = a.n_q_heads / a.n_kv_heads;
    const int Hkv = a.n_kv_heads;
    const float cscale = a.softmax_scale * 1.4426950408889634f;
    const uint32_t ring = __builtin_amdgcn_readfirstlane(lds_offset(smem)) + (uint32_t)(wave * NS * STAGE);
    const uint8_t *const ring_p = smem + wave * NS * STAGE;

    // LDS offsets inside a stage.  K operand: key m16, piece q4 + 4 kk.  V^T operand (transposing read): lane s of a
    // 16-lane group points at key 4 q4 + s / 4, dims 16 db + 4 (s % 4) .. and receives dim 16 db + s of keys 4 q4 .. + 3.
    const int k_rd = (m16 / KPC) * CH + (q4 * KPC + m16 % KPC) * 16;
    const int v_key = 4 * q4 + (m16 >> 2);
    const int v_rd = PAGE + (v_key / KPC) * CH + (((m16 & 3) >> 1) * KPC + v_key % KPC) * 16 + (m16 & 1) * 8;
    // loads: lane -> key lane % KPC of the chunk, piece lane / KPC
    const int ld_key = lane % KPC, ld_piece = lane / KPC;

    // constant rotation from a wavefront's page to its next one
    float2 step[KK / 2][8];
    const auto load_step = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < KK / 2; ++p) load_cs<D, STYLE>(a.rope, NWV * kPageSize, q4 + 4 * p, step[p]);
    };
    if (!ONE) load_step();

    const int it_end = ONE ? (int)blockIdx.x + 1 : load_uniform(a.wg_first + blockIdx.x + 1);
    for (int it = ONE ? (int)blockIdx.x : load_uniform(a.wg_first + blockIdx.x); it < it_end; ++it) {
        const int32_t *iw = reinterpret_cast<const int32_t *>(a.rows_items + it);
        // the ids of a wavefront's first pages are in the item (of sixteen pages in all)
        constexpr int NEAR = NS < 16 / NWV ? NS : 16 / NWV;
        int32_t near_page[NEAR];
#pragma unroll
        for (int s = 0; s < NEAR; ++s) near_page[s] = load_uniform(iw + 16 + wave + s * NWV);
        const int c = load_uniform(iw), g = load_uniform(iw + 1), n_rows = load_uniform(iw + 2);
        const int key_begin = load_uniform(iw + 3), key_end = load_uniform(iw + 4), part = load_uniform(iw + 5);
        const int n = load_uniform(iw + 6), q0 = load_uniform(iw + 7);
        const int32_t *table = a.block_table + (int64_t)c * a.max_pages;
        const int kmax = min(n + (n_rows - 1) / G + 1, key_end);       // exclusive end of the keys this item reads
        const int last_page = (kmax - 1) / kPageSize;
        int pg = key_begin / kPageSize + wave;

        auto issue = [&](int stage, int page_idx, int page) __attribute__((always_inline)) {
            const int64_t block = ((int64_t)page * Hkv + g) * kPageSize * D;
            const uint16_t *kb = a.k_pool + block, *vb = a.v_pool + block;
            const uint32_t at = ring + (uint32_t)(stage * STAGE);
            const int last_slot = kmax - 1 - page_idx * kPageSize;      // keys past the end: the last one again (finite data)
#pragma unroll
            for (int ch = 0; ch < CPP; ++ch) {
                const uint32_t off = (uint32_t)(min(ch * KPC + ld_key, last_slot) * D + ld_piece * 8) * 2u;
                dma16_sbase_nt(kb, off, at + ch * CH);
                dma16_sbase_nt(vb, off, at + PAGE + ch * CH);
            }
        };

        // ---- the first pages go out, then the query rows are fetched and rotated behind them -----------------------
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (pg + s * NWV <= last_page) issue(s, pg + s * NWV, s < NEAR ? near_page[s < NEAR ? s : 0] : load_uniform(table + pg + s * NWV));

        // Each row is fetched and rotated once per workgroup and handed on through LDS: a thread has one row's pair of pieces.
        for (int i = tid; i < n_rows * (PPR / 2); i += 64 * NWV) {
            const int r = i / (PPR / 2), piece = i % (PPR / 2), j = r / G;
            const uint16_t *qrow = a.q + ((int64_t)(q0 + j) * a.n_q_heads + g * G + (r - j * G)) * D;
            uint4 x = *reinterpret_cast<const uint4 *>(qrow + 8 * piece);
            uint4 y = *reinterpret_cast<const uint4 *>(qrow + HALF + 8 * piece);
            float2 qcs[8];
            load_cs<D, STYLE>(a.rope, n + j, piece, qcs);
            uint32_t *px = reinterpret_cast<uint32_t *>(&x), *py = reinterpret_cast<uint32_t *>(&y);
#pragma unroll
            for (int w = 0; w < 4; ++w) rotate_dword<STYLE>(px[w], py[w], qcs, w, cscale);
            *reinterpret_cast<uint4 *>(q_rot + r * QSTR + 16 * piece) = x;
            *reinterpret_cast<uint4 *>(q_rot + r * QSTR + D + 16 * piece) = y;
        }
        float2 cs[KK / 2][8];
#pragma unroll
        for (int p = 0; p < KK / 2; ++p) load_cs<D, STYLE>(a.rope, min(pg * kPageSize + m16, kmax - 1), q4 + 4 * p, cs[p]);
        if (ONE && pg + NWV <= last_page) load_step();
        int32_t next_page = load_uniform(table + min(pg + NS * NWV, last_page));      // id of the next page to ask for

        f32x4 O[NB][DB];
        float m_run[NB], l_run[NB];           // reference maximum of this lane's row (exponent units), its part of the denominator
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            m_run[nb] = -INFINITY;
            l_run[nb] = 0.f;
#pragma unroll
            for (int db = 0; db < DB; ++db) O[nb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        const bf16x2 ones2 = {(__bf16)1.0f, (__bf16)1.0f};

        // Everything the compiler loaded has arrived: it would otherwise wait for it at the first use inside the loop, every
        // time round, and with it for the pages just asked for.
        CA_WAIT_VMCNT(0);
        __syncthreads();
        bf16x8 Qf[NB][KK];
        int qpos[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int r = min(nb * 16 + m16, n_rows - 1);
            qpos[nb] = n + r / G;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) Qf[nb][kk] = *reinterpret_cast<const bf16x8 *>(q_rot + r * QSTR + 16 * (q4 + 4 * kk));
        }

        // ---- the walk ---------------------------------------------------------------------------------------------
        for (int stage = 0; pg <= last_page; pg += NWV, stage = (stage + 1) % NS) {
            // the pages behind this one may stay in flight
            if (pg + (NS - 1) * NWV <= last_page) { CA_WAIT_VMCNT((NS - 1) * LOADS); } else { CA_WAIT_VMCNT(0); }
            asm volatile("" : : : "memory");       // the reads stay behind the wait (no barrier says so here)
            const uint8_t *st = ring_p + stage * STAGE;
            uint4 k[KK];
            s16x4 v[DB];
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) k[kk] = *reinterpret_cast<const uint4 *>(st + k_rd + kk * (4 * KPC * 16));
#pragma unroll
            for (int db = 0; db < DB; ++db)
                v[db] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(st + v_rd + db * (2 * KPC * 16)));
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");       // read out: the stage is free
            if (pg + NS * NWV <= last_page) {
                issue(stage, pg + NS * NWV, next_page);
                next_page = load_uniform(table + min(pg + (NS + 1) * NWV, last_page));
            }

#pragma unroll
            for (int p = 0; p < KK / 2; ++p) {
                uint32_t *px = reinterpret_cast<uint32_t *>(&k[p]), *py = reinterpret_cast<uint32_t *>(&k[p + KK / 2]);
#pragma unroll
                for (int w = 0; w < 4; ++w) rotate_dword<STYLE>(px[w], py[w], cs[p], w);
                if (!ONE || pg + NWV <= last_page) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float2 o = cs[p][e], s = step[p][e];
                        cs[p][e] = make_float2(o.x * s.x - o.y * s.y, o.y * s.x + o.x * s.y);
                    }
                }
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const float nm = m_run[nb] == -INFINITY ? 0.f : -m_run[nb];
                f32x4 S = {nm, nm, nm, nm};
#pragma unroll
                for (int kk = 0; kk < KK; ++kk)
                    S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k[kk]), Qf[nb][kk], S, 0, 0, 0);
                const int key0 = pg * kPageSize + 4 * q4;
                if (pg * kPageSize + kPageSize - 1 > n) {               // some key of the page may be hidden from some row
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (key0 + i > qpos[nb]) S[i] = -INFINITY;
                }
                const float mx = fmaxf(fmaxf(S[0], S[1]), fmaxf(S[2], S[3]));
                const bool unseen = m_run[nb] == -INFINITY;
                if (__builtin_amdgcn_ballot_w64(mx > (unseen ? -INFINITY : kHeadroom)) != 0) {
                    const float all = over_row(mx, [](float x, float y) { return fmaxf(x, y); });
                    const bool raise = all > (unseen ? -INFINITY : kHeadroom);
                    const float delta = raise ? all : 0.f;
                    const float alpha = raise && !unseen ? __builtin_amdgcn_exp2f(-delta) : 1.0f;
                    if (raise) m_run[nb] = (unseen ? 0.f : m_run[nb]) + all;
                    l_run[nb] *= alpha;
#pragma unroll
                    for (int i = 0; i < 4; ++i) S[i] -= delta;
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int i = 0; i < 4; ++i) O[nb][db][i] *= alpha;
                }
                uint32_t pk[2];
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    pk[w] = pack_bf16(__builtin_amdgcn_exp2f(S[2 * w]), __builtin_amdgcn_exp2f(S[2 * w + 1]));
                    // the denominator sums the rounded probabilities, the very values the second product uses
                    l_run[nb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk[w]), ones2, l_run[nb], false);
                }
                const s16x4 pb = __builtin_bit_cast(s16x4, make_uint2(pk[0], pk[1]));
#pragma unroll
                for (int db = 0; db < DB; ++db) O[nb][db] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(v[db], pb, O[nb][db], 0, 0, 0);
            }
        }

        // ---- merge the wavefronts -----------------------------------------------------------------------------------
        __syncthreads();                       // the rings are free
        float *mo = reinterpret_cast<float *>(smem) + wave * ROWS * OSTR;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const float l = over_row(l_run[nb], [](float x, float y) { return x + y; });
            const int row = nb * 16 + m16;
            if (row < n_rows) {
#pragma unroll
                for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4 *>(mo + row * OSTR + db * 16 + 4 * q4) = O[nb][db];
                if (q4 == 0) {
                    red_m[wave][row] = m_run[nb];
                    red_l[wave][row] = l;
                }
            }
        }
        __syncthreads();
        constexpr int VPR = D / 4;
        // a share: [ROWS][D] sums, [ROWS] (maximum, denominator)
        constexpr int PART = ROWS * (D + 2) * 4;
        const auto shares = buffer_at(a.partial);
        for (int i = tid; i < n_rows * VPR; i += 64 * NWV) {
            const int row = i / VPR, d = 4 * (i % VPR);
            float M = red_m[0][row];
#pragma unroll
            for (int w = 1; w < NWV; ++w) M = fmaxf(M, red_m[w][row]);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            float l = 0.f;
#pragma unroll
            for (int w = 0; w < NWV; ++w) {
                const float f = red_m[w][row] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(red_m[w][row] - M);
                acc += f * *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(smem) + (w * ROWS + row) * OSTR + d);
                l += f * red_l[w][row];
            }
            if (part < 0) {
                store_out_row4<D>(a, q0, g, G, row, d, acc, 1.f / l);
            } else {
                store_agent4(shares, part * PART + (row * D + d) * 4, acc);
                if (d == 0) store_agent2(shares, part * PART + (ROWS * D + 2 * row) * 4, make_float2(M, l));
            }
        }
        if (part >= 0) {
            // the workgroup that brings a unit's last share merges them all
            const int ci = load_uniform(iw + 8), first = load_uniform(iw + 9), n_parts = load_uniform(iw + 10);
            if (arrive_last(a.arrived + ci, n_parts, &is_last)) {
                for (int i = tid; i < n_rows * VPR; i += 64 * NWV) {
                    const int row = i / VPR, d = 4 * (i % VPR);
                    float M = -INFINITY, l = 0.f;
                    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
                    constexpr int U = 8, BATCHES = ONE ? 2 : 1;         // shares of a batch, batches in flight
                    float2 ml0[U], ml1[U];                              // maximum, denominator
                    f32x4 os0[U], os1[U];
                    const auto fetch = [&](float2 (&ml)[U], f32x4 (&os)[U], int s0) __attribute__((always_inline)) {
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int at = (first + min(s0 + u, n_parts - 1)) * PART;
                            ml[u] = load_agent2(shares, at + (ROWS * D + 2 * row) * 4);
                            os[u] = load_agent4(shares, at + (row * D + d) * 4);
                        }
                    };
                    const auto add = [&](float2 (&ml)[U], const f32x4 (&os)[U], int s0) __attribute__((always_inline)) {
                        float M2 = M;
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            if (s0 + u >= n_parts) ml[u].x = -INFINITY;
                            M2 = fmaxf(M2, ml[u].x);
                        }
                        if (M2 == -INFINITY) return;
                        const float fa = __builtin_amdgcn_exp2f(M - M2);
                        acc *= fa;
                        l *= fa;
                        M = M2;
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const float fb = __builtin_amdgcn_exp2f(ml[u].x - M2);       // (0 where the share has seen no key)
                            if (ml[u].x != -INFINITY) acc += fb * os[u];
                            l += fb * (ml[u].x != -INFINITY ? ml[u].y : 0.f);
                        }
                    };
                    for (int s0 = 0; s0 < n_parts; s0 += BATCHES * U) {
                        fetch(ml0, os0, s0);
                        if (BATCHES == 2 && s0 + U < n_parts) fetch(ml1, os1, s0 + U);
                        add(ml0, os0, s0);
                        if (BATCHES == 2 && s0 + U < n_parts) add(ml1, os1, s0 + U);
                    }
                    store_out_row4<D>(a, q0, g, G, row, d, acc, 1.f / l);
                }
            }
        }
        __syncthreads();                       // the next item's loads overwrite the merge buffer
    }
}

template <int NB, int NWV, bool ONE>
hipError_t launch_blocks(const AttnArgs &a, hipStream_t stream) {
    const dim3 grid(a.n_wgs), block(64 * NWV);
    if (a.head_dim == 128 && a.rope_style == 0) hipLaunchKernelGGL((attn_rows_kernel<128, 0, NB, NWV, ONE>), grid, block, 0, stream, a);
    else if (a.head_dim == 128 && a.rope_style == 1) hipLaunchKernelGGL((attn_rows_kernel<128, 1, NB, NWV, ONE>), grid, block, 0, stream, a);
    else if (a.head_dim == 64 && a.rope_style == 0) hipLaunchKernelGGL((attn_rows_kernel<64, 0, NB, NWV, ONE>), grid, block, 0, stream, a);
    else if (a.head_dim == 64 && a.rope_style == 1) hipLaunchKernelGGL((attn_rows_kernel<64, 1, NB, NWV, ONE>), grid, block, 0, stream, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_rows(const AttnArgs &a, int wavefronts, bool runs, hipStream_t stream) {
    if (a.n_wgs <= 0) return hipSuccess;
    if (!a.wg_first || !a.rows_items || (a.n_combine > 0 && (!a.partial || !a.arrived))) return hipErrorInvalidValue;
    if (a.tile_rows == 16) return runs ? launch_blocks<1, 4, false>(a, stream) : wavefronts == 8 ? launch_blocks<1, 8, true>(a, stream) : launch_blocks<1, 4, true>(a, stream);
    if (a.tile_rows == 32) return runs ? launch_blocks<2, 4, false>(a, stream) : wavefronts == 8 ? launch_blocks<2, 8, true>(a, stream) : launch_blocks<2, 4, true>(a, stream);
    return hipErrorInvalidValue;
}

}  // namespace ca
