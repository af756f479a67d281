// Data-movement kernels of the layer-wise load / save path (Section 3.2) and the per-token
// metadata of the rebased plan (Section 3.4).  Pure integer indexing and 16-byte copies:
// results are bit-exact by construction.
//
// HBM-bound.  Per token and layer the kernels move n_kv_heads*head_dim*2 bytes of K and as many
// of V, read once and written once.  For a fixed head, 16 consecutive context tokens are one whole
// (page, head) block of the pool (4 KiB contiguous) on the paged side and 16 rows of 256 B on the
// contiguous side, so both sides move in full 256-byte segments; all heads of a page together are
// one contiguous run on either side (n_kv_heads * 4 KiB in the pool, 16 whole token rows in the
// contiguous layout).
#include "ca_device.h"
#include "ca_internal.h"

namespace ca {

namespace {

typedef __attribute__((ext_vector_type(4))) unsigned int vec16;  // one 16-byte piece

constexpr int kMoveThreads = 256;
constexpr int kUnroll = kMoveUnroll;
constexpr int kMoveMaxGridY = 32768;


// One contiguous range of context tokens of one conversation, for keys or for values, and where it lies outside the pool.
struct Piece {
    uint8_t *contig;        // token contig_tok0 + i <-> context token ctx_tok0 + i, i < count
    int64_t contig_tok0;
    int ctx_tok0, count, seq;
    uint8_t *second;        // kDual: row i receives token i too
};

// grid: x = (slice of heads, K or V), y = page of the conversation's context (counted from the first
// page the range touches), z = conversation entry of this launch.  A workgroup moves, for one of the
// two arrays, the tokens of its page that lie inside the range for heads_per_wg heads, kUnroll loads
// of 16 bytes in flight per lane before the first store.  The page id is uniform over the workgroup.
// The order matters: x is the fastest launch dimension, so the workgroups that together cover one
// page run next to each other and both sides of the copy see long sequential runs; with few loads
// in flight per lane and keys and values in separate workgroups the kernel reaches 5.7 TB/s on a
// 337 MB load where the opposite choices (pages fastest, 4 + 4 loads per lane) gave 5.0.
// kDual (with kToPool): every vector read from the contiguous side is stored twice, into the pool and into a second
// contiguous destination (the tier): the new turn's K/V are appended and saved in one pass over them.
template <bool kToPool, bool kNT, bool kDual>
__device__ inline void move_piece(const Piece &p, const MoveShape &s, uint8_t *__restrict__ side) {
    static_assert(!kDual || kToPool, "the second destination goes with contiguous -> pages");
    const int ctx_begin = p.ctx_tok0;
    const int ctx_end = ctx_begin + p.count;
    const int vs = s.vec_shift;
    // grid.y is capped below the launch limit; longer ranges take more than one trip
    for (int col = blockIdx.y; col < s.max_pages_touched; col += gridDim.y) {
        const int page_col = ctx_begin / kPageSize + col;
        const int t_first = max(ctx_begin, page_col * kPageSize);
        const int t_last = min(ctx_end, (page_col + 1) * kPageSize);   // exclusive
        if (t_first >= t_last) break;   // past the last page of this range
        const int slot0 = t_first - page_col * kPageSize;
        const int n_tok = t_last - t_first;
        const int H = s.n_kv_heads;
        const int h_first = (blockIdx.x >> 1) * s.heads_per_wg;
        const int h_count = min(s.heads_per_wg, H - h_first);
        const int page = load_uniform(s.block_table + (int64_t)p.seq * s.max_pages + page_col);
        const int64_t row_vecs = (int64_t)H << vs;  // 16-byte vectors per token on the contiguous side
        const int64_t contig_first = p.contig_tok0 + (t_first - ctx_begin);
        vec16 *contig = reinterpret_cast<vec16 *>(p.contig) + contig_first * row_vecs + ((int64_t)h_first << vs);
        vec16 *pool = reinterpret_cast<vec16 *>(side) + ((((int64_t)page * H + h_first) * kPageSize + slot0) << vs);
        vec16 *second = nullptr;
        if (kDual) second = reinterpret_cast<vec16 *>(p.second) + (t_first - ctx_begin) * row_vecs + ((int64_t)h_first << vs);

        // vector id v -> (head, token, 16-byte piece), piece fastest
        const int per_head = n_tok << vs;
        const int total = h_count * per_head;
        for (int v0 = threadIdx.x; v0 < total; v0 += kMoveThreads * kUnroll) {
            vec16 r[kUnroll];
            int pool_idx[kUnroll];
            int64_t contig_idx[kUnroll];
            bool live[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int v = v0 + u * kMoveThreads;
                const int hl = n_tok == kPageSize ? v / kPageSize >> vs : v / per_head;
                const int rem = v - hl * per_head;
                const int ti = rem >> vs;
                const int piece = rem - (ti << vs);
                live[u] = v < total;
                pool_idx[u] = (((hl * kPageSize) + ti) << vs) + piece;
                contig_idx[u] = (int64_t)ti * row_vecs + (hl << vs) + piece;
                if (live[u]) {
                    const vec16 *src = kToPool ? contig + contig_idx[u] : pool + pool_idx[u];
                    r[u] = kNT ? __builtin_nontemporal_load(src) : *src;
                }
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if (live[u]) {
                    vec16 *dst = kToPool ? pool + pool_idx[u] : contig + contig_idx[u];
                    if (kNT) __builtin_nontemporal_store(r[u], dst); else *dst = r[u];
                    if (kDual) __builtin_nontemporal_store(r[u], second + contig_idx[u]);
                }
            }
        }
    }
}

template <bool kToPool, bool kNT>
__global__ __launch_bounds__(kMoveThreads) void move_kernel(MoveArgs a, MoveShape s, uint8_t *__restrict__ k_pool,
                                                            uint8_t *__restrict__ v_pool) {
    const int e = blockIdx.z;  // entry of this launch
    const bool values = blockIdx.x & 1;
    const Piece p{values ? a.contig_v[e] : a.contig_k[e], a.contig_tok0[e], a.ctx_tok0[e], a.count[e], a.seq[e], nullptr};
    move_piece<kToPool, kNT, false>(p, s, values ? v_pool : k_pool);
}

// Moves between the pool and pinned host memory: bound by the host link, which a few workgroups keep full (a round trip
// takes about 2 us and a workgroup has 32 KB in flight; 8 to 10 of them read at 57 GB/s, which is what one large copy by a
// copy engine reaches).  A grid that filled the GPU with waiting wavefronts holds up the kernels running beside it; so do
// loads issued ahead of the stores (with 8 workgroups the attention beside a load 1.25 x instead of 1.07 x, the load no
// faster).  A workgroup's unit is a group of consecutive pages of one conversation, keys or values: whole token rows,
// contiguous on the host side, about 32 KB (one page of 8 heads of 128 or more).  first[e] = groups of the entries before e.
struct LinkUnits {
    int32_t first[kMaxSeqsPerLaunch + 1];
    int32_t pages;        // pages per group
};

template <bool kToPool, bool kOnePage>      // kOnePage: units.pages == 1, the page is uniform over the workgroup
__global__ __launch_bounds__(kMoveThreads) void link_kernel(MoveArgs a, LinkUnits units, MoveShape s, uint8_t *__restrict__ k_pool,
                                                            uint8_t *__restrict__ v_pool) {
    constexpr int kLinkUnroll = 8;
    const int vs = s.vec_shift;
    const int H = s.n_kv_heads;
    const int row_vecs = H << vs;
    const bool values = blockIdx.x & 1;
    vec16 *const side = reinterpret_cast<vec16 *>(values ? v_pool : k_pool);
    const int n_units = units.first[s.n_in_launch];
    int e = 0;
    for (int unit = blockIdx.x >> 1; unit < n_units; unit += gridDim.x >> 1) {
        while (unit >= units.first[e + 1]) ++e;
        const int begin = a.ctx_tok0[e], end = begin + a.count[e];
        const int page_col = begin / kPageSize + (unit - units.first[e]) * units.pages;
        const int t_first = max(begin, page_col * kPageSize), t_last = min(end, (page_col + units.pages) * kPageSize);
        const int total = (t_last - t_first) * row_vecs;
        const int32_t *table = s.block_table + (int64_t)a.seq[e] * s.max_pages + page_col;
        vec16 *contig = reinterpret_cast<vec16 *>(values ? a.contig_v[e] : a.contig_k[e]) + (a.contig_tok0[e] + (t_first - begin)) * row_vecs;
        // page ids of the unit: one (by a scalar load, which no store is waited for with), or page i in lane i of every wavefront
        const int pages = kOnePage ? load_uniform(table) : table[min((int)threadIdx.x & 63, (t_last - 1) / kPageSize - page_col)];
        for (int v0 = threadIdx.x; v0 - (int)threadIdx.x < total; v0 += kMoveThreads * kLinkUnroll) {
            // where vector v of the unit lies in the pool
            const auto in_pool = [&](int v) __attribute__((always_inline)) {
                const int row = v / row_vecs;
                const int rem = v - row * row_vecs;       // (head, piece)
                const int slot = t_first + row - page_col * kPageSize;
                const int page = kOnePage ? pages : __shfl(pages, slot / kPageSize);
                return side + (((((int64_t)page * H + (rem >> vs)) * kPageSize + slot % kPageSize) << vs) + (rem & ((1 << vs) - 1)));
            };
            // loads without conditions, back to back (past the end: the last vector again, not stored)
            vec16 r[kLinkUnroll];
#pragma unroll
            for (int u = 0; u < kLinkUnroll; ++u) {
                const int v = min(v0 + u * kMoveThreads, total - 1);
                r[u] = __builtin_nontemporal_load(kToPool ? contig + v : in_pool(v));
            }
            // All of them before the first store: the compiler then sees no load outstanding at the head of the loop and puts
            // no wait there, which would be one for the stores as well (45 GB/s with 8 workgroups instead of 57).
            __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
            for (int u = 0; u < kLinkUnroll; ++u) {
                const int v = min(v0 + u * kMoveThreads, total - 1);
                vec16 *dst = kToPool ? in_pool(v) : contig + v;
                if (v0 + u * kMoveThreads < total) __builtin_nontemporal_store(r[u], dst);
            }
        }
    }
}

// The new turn of conversation `seq`: everything but the pointers is in the plan's metadata, so the arguments are a few
// words whatever the batch (a launch with 2.6 KB of per-conversation arguments costs the host 0.4 to 1.3 us more).
__device__ inline Piece new_turn(const MoveShape &s, int seq, const uint8_t *from, uint8_t *second) {
    const int q = load_uniform(s.cu_q + seq);
    return Piece{const_cast<uint8_t *>(from), q, load_uniform(s.n_keep + seq), load_uniform(s.cu_q + seq + 1) - q, seq, second};
}

__global__ __launch_bounds__(kMoveThreads) void append_kernel(MoveShape s, const uint8_t *__restrict__ new_k, const uint8_t *__restrict__ new_v,
                                                              uint8_t *__restrict__ k_pool, uint8_t *__restrict__ v_pool) {
    const bool values = blockIdx.x & 1;
    move_piece<true, true, false>(new_turn(s, blockIdx.z, values ? new_v : new_k, nullptr), s, values ? v_pool : k_pool);
}

__global__ __launch_bounds__(kMoveThreads) void append_save_kernel(MoveArgs2 b, MoveShape s, int first, const uint8_t *__restrict__ new_k,
                                                                   const uint8_t *__restrict__ new_v, uint8_t *__restrict__ k_pool,
                                                                   uint8_t *__restrict__ v_pool) {
    const bool values = blockIdx.x & 1;
    move_piece<true, true, true>(new_turn(s, first + blockIdx.z, values ? new_v : new_k, values ? b.dst_v[blockIdx.z] : b.dst_k[blockIdx.z]), s,
                                 values ? v_pool : k_pool);
}

// A token's keys (or values) between a contiguous row and its slot of the pool: grid (slices of 256 vectors x {K, V}, token).
// Such a move is a chain of dependent accesses and nothing else: with conversation, position and page looked up one after
// the other (append_kernel, move_kernel) a decode step's append and save took 4.7 us each for 16 conversations of 32 heads;
// here the arguments bring the slot and the first access is the data itself.  A decode step of one conversation (64/8 heads,
// 2777 tokens, 80 layers) went from 1585 to 1515 us, one of 16 conversations (32 heads, 32 layers) from 1978 to 1942.
template <bool kToPool>
__device__ inline void move_token(int slot, int H, int vs, uint8_t *row, uint8_t *pool) {
    const int v = (blockIdx.x >> 1) * kMoveThreads + threadIdx.x;
    if (v >= H << vs) return;
    vec16 *const in_row = reinterpret_cast<vec16 *>(row) + v;
    vec16 *const in_pool = reinterpret_cast<vec16 *>(pool) +
                           (((((int64_t)(slot / kPageSize) * H + (v >> vs)) * kPageSize + slot % kPageSize) << vs) + (v & ((1 << vs) - 1)));
    if (kToPool) __builtin_nontemporal_store(__builtin_nontemporal_load(in_row), in_pool);
    else __builtin_nontemporal_store(__builtin_nontemporal_load(in_pool), in_row);
}

__global__ __launch_bounds__(kMoveThreads) void append_tokens_kernel(TokenSlots t, int H, int vs, const uint8_t *__restrict__ new_k,
                                                                     const uint8_t *__restrict__ new_v, uint8_t *__restrict__ k_pool,
                                                                     uint8_t *__restrict__ v_pool) {
    const bool values = blockIdx.x & 1;
    const uint8_t *row = (values ? new_v : new_k) + (((int64_t)blockIdx.y * H << vs) * sizeof(vec16));
    move_token<true>(t.slot[blockIdx.y], H, vs, const_cast<uint8_t *>(row), values ? v_pool : k_pool);
}

__global__ __launch_bounds__(kMoveThreads) void save_tokens_kernel(TokenSlots t, TokenRows r, int H, int vs, uint8_t *__restrict__ k_pool,
                                                                   uint8_t *__restrict__ v_pool) {
    const bool values = blockIdx.x & 1;
    move_token<false>(t.slot[blockIdx.y], H, vs, values ? r.v[blockIdx.y] : r.k[blockIdx.y], values ? v_pool : k_pool);
}

// Brings a plan's metadata to the device and forms its per-token arrays, in one launch and without a copy engine: the
// image is read from pinned host memory by the kernel (20 KB: 3 us, where hipMemcpyAsync in front of a kernel took 15 to
// 35 us).  The first copy_wgs workgroups copy; the others own 256 context tokens of one conversation at a time: where a token
// lives in the pool, and for new tokens their rebased position.  They read what they need of the image from the host as
// well, two dependent reads, so nothing waits for the copy inside the launch.
constexpr int kRebaseThreads = 256;
__global__ __launch_bounds__(kRebaseThreads) void rebase_kernel(RebaseArgs a, int copy_wgs, int chunks) {
    if ((int)blockIdx.x < copy_wgs) {
        const vec16 *src = reinterpret_cast<const vec16 *>(a.image);
        vec16 *dst = reinterpret_cast<vec16 *>(a.meta);
        for (int64_t i = (int64_t)blockIdx.x * kRebaseThreads + threadIdx.x; i < a.image_vecs; i += (int64_t)copy_wgs * kRebaseThreads) dst[i] = src[i];
        for (int i = blockIdx.x * kRebaseThreads + threadIdx.x; i < a.n_merges; i += copy_wgs * kRebaseThreads) a.arrived[0][i] = a.arrived[1][i] = 0;
        return;
    }
    const int at = blockIdx.x - copy_wgs;
    const int c = at / chunks;
    const int32_t *cu_k = reinterpret_cast<const int32_t *>(a.image + a.off_cu_k);
    const int k0 = cu_k[c], len = cu_k[c + 1] - k0;
    const int n = reinterpret_cast<const int32_t *>(a.image + a.off_n_keep)[c];
    const int q0 = reinterpret_cast<const int32_t *>(a.image + a.off_cu_q)[c];
    for (int t = (at - c * chunks) * kRebaseThreads + threadIdx.x; t < len; t += chunks * kRebaseThreads) {
        const int page = reinterpret_cast<const int32_t *>(a.image + a.off_table)[(int64_t)c * a.max_pages + t / kPageSize];
        a.slot_map[k0 + t] = page * kPageSize + t % kPageSize;
        if (t >= n) {
            a.q_pos[q0 + t - n] = t;  // new token j sits at position n + j of the truncated context
            a.q_seq[q0 + t - n] = c;
        }
    }
}

}  // namespace

hipError_t launch_move(bool to_pool, const MoveArgs &args, const MoveShape &shape, uint8_t *k_pool,
                       uint8_t *v_pool, hipStream_t stream) {
    if (shape.n_in_launch <= 0 || shape.max_pages_touched <= 0) return hipSuccess;
    const int slices = (shape.n_kv_heads + shape.heads_per_wg - 1) / shape.heads_per_wg;
    const int rows = std::min(shape.max_pages_touched, kMoveMaxGridY);
    dim3 grid(2 * slices, rows, shape.n_in_launch);
    // nontemporal accesses: every byte is touched once (measured ~5 % faster than cached ones)
    if (to_pool)
        hipLaunchKernelGGL((move_kernel<true, true>), grid, dim3(kMoveThreads), 0, stream, args, shape, k_pool, v_pool);
    else
        hipLaunchKernelGGL((move_kernel<false, true>), grid, dim3(kMoveThreads), 0, stream, args, shape, k_pool, v_pool);
    return hipGetLastError();
}

hipError_t launch_link(bool to_pool, const MoveArgs &args, const MoveShape &shape, int workgroups, uint8_t *k_pool, uint8_t *v_pool,
                       hipStream_t stream) {
    LinkUnits units;
    units.pages = std::max(1, std::min(64, 2048 / ((kPageSize * shape.n_kv_heads) << shape.vec_shift)));     // 2048 vectors = 32 KB
    units.first[0] = 0;
    for (int i = 0; i < shape.n_in_launch; ++i) {
        const int pages = args.count[i] > 0 ? (args.ctx_tok0[i] + args.count[i] - 1) / kPageSize - args.ctx_tok0[i] / kPageSize + 1 : 0;
        units.first[i + 1] = units.first[i] + (pages + units.pages - 1) / units.pages;
    }
    const int n = units.first[shape.n_in_launch];
    if (n <= 0) return hipSuccess;
    const dim3 grid(2 * std::min(n, std::max(1, workgroups / 2)));
    const auto kernel = to_pool ? (units.pages == 1 ? link_kernel<true, true> : link_kernel<true, false>)
                                : (units.pages == 1 ? link_kernel<false, true> : link_kernel<false, false>);
    hipLaunchKernelGGL(kernel, grid, dim3(kMoveThreads), 0, stream, args, units, shape, k_pool, v_pool);
    return hipGetLastError();
}

hipError_t launch_append(const MoveShape &shape, const uint8_t *new_k, const uint8_t *new_v, uint8_t *k_pool, uint8_t *v_pool,
                         hipStream_t stream) {
    if (shape.n_in_launch <= 0 || shape.max_pages_touched <= 0) return hipSuccess;
    const int slices = (shape.n_kv_heads + shape.heads_per_wg - 1) / shape.heads_per_wg;
    dim3 grid(2 * slices, std::min(shape.max_pages_touched, kMoveMaxGridY), shape.n_in_launch);
    hipLaunchKernelGGL(append_kernel, grid, dim3(kMoveThreads), 0, stream, shape, new_k, new_v, k_pool, v_pool);
    return hipGetLastError();
}

hipError_t launch_append_save(const MoveShape &shape, int first, const MoveArgs2 &second, const uint8_t *new_k, const uint8_t *new_v,
                              uint8_t *k_pool, uint8_t *v_pool, hipStream_t stream) {
    if (shape.n_in_launch <= 0 || shape.max_pages_touched <= 0) return hipSuccess;
    const int slices = (shape.n_kv_heads + shape.heads_per_wg - 1) / shape.heads_per_wg;
    dim3 grid(2 * slices, std::min(shape.max_pages_touched, kMoveMaxGridY), shape.n_in_launch);
    hipLaunchKernelGGL(append_save_kernel, grid, dim3(kMoveThreads), 0, stream, second, shape, first, new_k, new_v, k_pool, v_pool);
    return hipGetLastError();
}

hipError_t launch_append_tokens(const TokenSlots &slots, int n, const MoveShape &shape, const uint8_t *new_k, const uint8_t *new_v,
                                uint8_t *k_pool, uint8_t *v_pool, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const dim3 grid(2 * (((shape.n_kv_heads << shape.vec_shift) + kMoveThreads - 1) / kMoveThreads), n);
    hipLaunchKernelGGL(append_tokens_kernel, grid, dim3(kMoveThreads), 0, stream, slots, shape.n_kv_heads, shape.vec_shift, new_k, new_v, k_pool, v_pool);
    return hipGetLastError();
}

hipError_t launch_save_tokens(const TokenSlots &slots, const TokenRows &rows, int n, const MoveShape &shape, const uint8_t *k_pool,
                              const uint8_t *v_pool, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const dim3 grid(2 * (((shape.n_kv_heads << shape.vec_shift) + kMoveThreads - 1) / kMoveThreads), n);
    hipLaunchKernelGGL(save_tokens_kernel, grid, dim3(kMoveThreads), 0, stream, slots, rows, shape.n_kv_heads, shape.vec_shift,
                       const_cast<uint8_t *>(k_pool), const_cast<uint8_t *>(v_pool));
    return hipGetLastError();
}

hipError_t launch_rebase(const RebaseArgs &args, hipStream_t stream) {
    if (args.n_seqs <= 0) return hipSuccess;
    const int chunks = std::min((args.max_pages * kPageSize + kRebaseThreads - 1) / kRebaseThreads, std::max(1, (1 << 20) / args.n_seqs));
    const int copy_wgs = (int)std::max<int64_t>(1, std::min<int64_t>(256, (args.image_vecs + kRebaseThreads - 1) / kRebaseThreads));
    hipLaunchKernelGGL(rebase_kernel, dim3(copy_wgs + chunks * args.n_seqs), dim3(kRebaseThreads), 0, stream, args, copy_wgs, chunks);
    return hipGetLastError();
}

}  // namespace ca
