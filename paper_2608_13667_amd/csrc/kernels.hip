// HIP kernels for fork-aware decode attention on gfx950 (CDNA4, wave64).
//
// (the partial-attention kernel over key ranges lives in partials.hip)
// merge_kernel: log-sum-exp combination of the partials of each (sequence, head).
// append_kernel / gather_kernel: suffix append and paged gather (data movement).
#include "internal.h"
#include "merge_row.h"

namespace fka {
namespace {

// Where a row's parts are: kExplicit, every row merges parts 0 .. n_parts-1; a plan's split, even
// (whole blocks per item), or the general static one or the proportional one.
enum class MergeParts { kExplicit, kEven, kPlan };

// Fused step, block (Hq, seq): stores the token the sequence appends (the merging blocks attend to it
// from k_new / v_new) and advances suffix_len[seq].  No block of the merge reads the suffix
// cache or suffix_len (the lengths come from the partial kernel), so nothing races.  A block of its own,
// because the page look-up behind the length would make a merging block the launch's last.
template <int HD>
__device__ inline void append_token(const MergeArgs &a, int seq)
{
    constexpr int APP = HD / 8;  // 16-byte chunks of one K/V row
    const int tid = threadIdx.x;
    // the length, the prefix length and the first 256 chunks on their way together: as vector loads,
    // since scalar ones would be waited for one by one
    int zero = 0;
    asm("" : "+v"(zero));
    const int L = a.lens[seq + zero];
    int plen = 0;
    if (a.paged) plen = a.seq_prefix_len[seq + zero];
    uint4 app_k = {0, 0, 0, 0}, app_v = {0, 0, 0, 0};
    if (tid < a.n_kv_heads * APP) {
        const size_t src = (size_t)seq * a.n_kv_heads * HD + 8 * tid;
        app_k = *reinterpret_cast<const uint4 *>(a.k_new + src);
        app_v = *reinterpret_cast<const uint4 *>(a.v_new + src);
    }
    bool ok = L < a.max_suffix_len;
    int page = 0;
    if (a.paged) {
        const int pidx = (plen + kPageSize - 1) / kPageSize + L / kPageSize;
        page = ok && pidx < a.max_pages ? a.page_table[(size_t)seq * a.max_pages + pidx] : -1;
        ok = page >= 0 && page < a.n_pool_pages;
    }
    if (ok) {
        for (int c = tid; c < a.n_kv_heads * APP; c += 256) {
            const int gg = c / APP, cc = c % APP;
            const size_t dst =
                a.paged ? (((size_t)page * a.n_kv_heads + gg) * kPageSize + L % kPageSize) * HD + 8 * cc
                        : (((size_t)seq * a.n_kv_heads + gg) * a.suffix_cap + L) * HD + 8 * cc;
            uint4 kk = app_k, vv = app_v;
            if (c >= 256) {
                const size_t src = ((size_t)seq * a.n_kv_heads + gg) * HD + 8 * cc;
                kk = *reinterpret_cast<const uint4 *>(a.k_new + src);
                vv = *reinterpret_cast<const uint4 *>(a.v_new + src);
            }
            *reinterpret_cast<uint4 *>(a.k_dst + dst) = kk;
            *reinterpret_cast<uint4 *>(a.v_dst + dst) = vv;
        }
    }
    if (tid == 0) {
        if (ok)
            a.suffix_len[seq] = L + 1;
        else
            atomicOr(a.err, kErrAppendNoRoom);
    }
}

// One block per output row (plan modes: block (query head, sequence), so that neither needs a division).
// A kernel for each way to find the parts and for the step, so that a launch reads its arguments at
// once and waits for nothing in front of the part loads (one kernel for all of them waited for the
// length, for q and the appended key, and for arguments read late: a fused step at 8k keys took 18.2 us, now 16.9,
// at 512 keys and d 64 11.5, now 10.4).
template <int HD, MergeParts PARTS, bool STEP>
__global__ __launch_bounds__(256) void merge_kernel(MergeArgs a)
{
    __shared__ MergeLds<HD> lds;
    // the arguments in one go (the compiler would load some of them only where they are used, a scalar
    // load behind the other)
    asm volatile("" ::"s"(a.part_o), "s"(a.part_lse), "s"(a.out), "s"(a.out_lse), "s"(a.n_q_heads));
    if constexpr (PARTS == MergeParts::kExplicit) asm volatile("" ::"s"(a.rows), "s"(a.n_parts));
    if constexpr (PARTS != MergeParts::kExplicit)
        asm volatile("" ::"s"(a.slot_rows), "s"(a.group), "s"(a.group_magic), "s"(a.even_bpi), "s"(a.rowrec));
    if constexpr (STEP)
        asm volatile("" ::"s"(a.lens), "s"(a.q), "s"(a.k_new), "s"(a.v_new), "s"(a.scale), "s"(a.n_kv_heads),
                     "s"(a.max_suffix_len), "s"(a.seq_prefix_len), "s"(a.page_table));
    RowMerge m{};
    m.part_o = a.part_o;
    m.part_lse = a.part_lse;
    int row = blockIdx.x;
    if constexpr (PARTS == MergeParts::kExplicit) {
        m.n = a.n_parts;
        m.p_first = row;
        m.p_step = a.rows;
    } else {
        const int h = blockIdx.x, seq = blockIdx.y;
        if (STEP && h == a.n_q_heads) {
            append_token<HD>(a, seq);
            return;
        }
        row = seq * a.n_q_heads + h;
        const int g = div_magic(h, a.group, a.group_magic);
        m.p_step = a.slot_rows;
        if constexpr (PARTS == MergeParts::kEven) {  // item g's blocks g bpi .. write slots vb + g
            m.n = a.even_bpi;
            m.p_first = (uint32_t)(g * a.even_bpi + g) * a.slot_rows + seq * a.group + (h - g * a.group);
        } else if (a.static_split) {
            // item g owns workers [floor(g NV / Hkv), floor((g+1) NV / Hkv)); its blocks write
            // their partials to slots vb + g; the one unit starts at sequence 0
            const int ws0 = static_start(g, a.n_workers, a.n_kv_heads);
            const int ws1 = static_start(g + 1, a.n_workers, a.n_kv_heads);
            const int vb0 = ws0 / a.waves;
            m.n = ws1 > ws0 ? (ws1 - 1) / a.waves - vb0 + 1 : 0;
            m.p_first = (uint32_t)(vb0 + g) * a.slot_rows + seq * a.group + (h - g * a.group);
        } else {
            const int2 rec = *reinterpret_cast<const int2 *>(a.rowrec + (size_t)row * kRowRec);
            // a record that points outside the workspace (it cannot, unless the workspace was
            // overwritten from outside) is dropped and flagged rather than followed
            const int64_t lim = (int64_t)a.n_slots * a.slot_rows;
            const bool ok = rec.y >= 0 && rec.x >= 0 && (int64_t)rec.x + (int64_t)max(rec.y - 1, 0) * a.slot_rows < lim;
            if (!ok && threadIdx.x == 0) atomicOr(a.err, kErrBadSchedule);
            m.p_first = rec.x;
            m.n = ok ? rec.y : 0;
        }
        if constexpr (STEP) {
            m.len = a.lens + seq;
            m.max_len = a.max_suffix_len;
            m.q_row = a.q + (size_t)row * HD;
            m.k_row = a.k_new + ((size_t)seq * a.n_kv_heads + g) * HD;
            m.v_row = a.v_new + ((size_t)seq * a.n_kv_heads + g) * HD;
            m.scale = a.scale;
        }
    }
    m.out_row = a.out + (size_t)row * HD;
    m.out_lse = a.out_lse ? a.out_lse + row : nullptr;
    merge_row<HD, STEP>(m, lds);
}

// The explicit-mode merge for many rows of few parts (the tiled prefill's): HD / 4 lanes per row, each
// holding four floats of it, so a block of 256 threads merges 8 (d = 128) or 16 rows and every
// thread has up to eight parts in flight.  (One block per row keeps eight part slices of threads
// apart, most of them idle with the 4-16 parts of a prefill.)  Bound: the parts' bytes, from L2 and
// the Infinity Cache where the prefill kernel left them.
constexpr int kMergeBatch = 8;

template <int HD>
__global__ __launch_bounds__(256) void merge_rows_kernel(MergeArgs a)
{
    constexpr int CH = HD / 4;
    constexpr float kLog2eM = 1.442695040888963407f;
    const int chunk = threadIdx.x % CH, row = (int)blockIdx.x * (256 / CH) + threadIdx.x / CH;
    if (row >= a.rows) return;
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc((void *)a.part_o, 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc((void *)a.part_lse, 0, 0x7fffffff, 0x00020000);
    float M = -INFINITY, W = 0.f;
    merge_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0; j0 < a.n_parts; j0 += kMergeBatch) {
        float l[kMergeBatch];
        merge_f32x4 o[kMergeBatch];
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u) {
            l[u] = -INFINITY;
            o[u] = merge_f32x4{0.f, 0.f, 0.f, 0.f};
            if (j0 + u < a.n_parts) {
                const uint32_t part = (uint32_t)(j0 + u) * (uint32_t)a.rows + (uint32_t)row;
                l[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rl, part * 4, 0, 0));
                o[u] = __builtin_bit_cast(merge_f32x4, __builtin_amdgcn_raw_buffer_load_b128(ro, part * (HD * 4) + 16 * chunk, 0, 0));
            }
        }
        float Mn = M;
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u) Mn = fmaxf(Mn, l[u]);
        const float Mu = (Mn == -INFINITY) ? 0.f : Mn;
        const float sc = (M == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f((M - Mu) * kLog2eM);
        W *= sc;
        acc *= sc;
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u) {
            if (l[u] == -INFINITY) continue;  // an empty part's o is not read
            const float e = __builtin_amdgcn_exp2f((l[u] - Mu) * kLog2eM);
            W += e;
            acc += e * o[u];
        }
        M = Mn;
    }
    const merge_f32x4 r = (W == 0.f) ? merge_f32x4{0.f, 0.f, 0.f, 0.f} : acc * __builtin_amdgcn_rcpf(W);
    *reinterpret_cast<merge_f32x4 *>(a.out + (size_t)row * HD + 4 * chunk) = r;
    if (a.out_lse && chunk == 0) a.out_lse[row] = (W == 0.f) ? -INFINITY : ((M == -INFINITY) ? 0.f : M) + logf(W);
}

__global__ __launch_bounds__(256) void append_kernel(AppendArgs a)
{
    const int seq = blockIdx.x;
    __shared__ int s_row, s_page;
    if (threadIdx.x == 0) {
        const int L = a.suffix_len[seq];
        bool ok = L >= 0 && L < a.max_suffix_len;
        int page = 0;
        if (ok && a.paged) {
            const int lp = a.seq_prefix_len[seq];
            const int pidx = (lp + kPageSize - 1) / kPageSize + L / kPageSize;
            page = pidx < a.max_pages ? a.page_table[(size_t)seq * a.max_pages + pidx] : -1;
            ok = page >= 0 && page < a.n_pool_pages;
        }
        if (!ok) atomicOr(a.err, kErrAppendNoRoom);
        s_row = ok ? L : -1;
        s_page = page;
    }
    __syncthreads();
    const int row = s_row;
    if (row < 0) return;
    const int cpr = a.head_dim / 8;
    const int chunks = a.n_kv_heads * cpr;
    for (int c = threadIdx.x; c < chunks; c += blockDim.x) {
        const int g = c / cpr, cc = c % cpr;
        const size_t src = ((size_t)seq * a.n_kv_heads + g) * a.head_dim + 8 * cc;
        size_t dst;
        if (a.paged)
            dst = (((size_t)s_page * a.n_kv_heads + g) * kPageSize + row % kPageSize) * a.head_dim + 8 * cc;
        else
            dst = (((size_t)seq * a.n_kv_heads + g) * a.suffix_cap + row) * a.head_dim + 8 * cc;
        *reinterpret_cast<uint4 *>(a.k_dst + dst) = *reinterpret_cast<const uint4 *>(a.k_new + src);
        *reinterpret_cast<uint4 *>(a.v_dst + dst) = *reinterpret_cast<const uint4 *>(a.v_new + src);
    }
    __syncthreads();
    if (threadIdx.x == 0) a.suffix_len[seq] = row + 1;
}

// grid (ceil((out_len - begin) / 16), Hkv): block copies 16 logical positions of one KV head.
__global__ __launch_bounds__(256) void gather_kernel(GatherArgs a)
{
    const int g = blockIdx.y;
    const int cpr = a.head_dim / 8;
    for (int i = threadIdx.x; i < kPageSize * cpr; i += blockDim.x) {
        const int pos = a.begin + blockIdx.x * kPageSize + i / cpr, c = i % cpr;
        if (pos >= a.out_len) continue;
        int pidx, slot;
        if (pos < a.prefix_len) {
            pidx = pos / kPageSize;
            slot = pos % kPageSize;
        } else {
            const int u = pos - a.prefix_len;
            pidx = (a.prefix_len + kPageSize - 1) / kPageSize + u / kPageSize;
            slot = u % kPageSize;
        }
        const int page = a.page_table[(size_t)a.seq * a.max_pages + pidx];
        const size_t dst = ((size_t)g * (a.out_len - a.begin) + (pos - a.begin)) * a.head_dim + 8 * c;
        uint4 kv = uint4{0, 0, 0, 0}, vv = uint4{0, 0, 0, 0};
        if (page >= 0 && page < a.n_pool_pages) {
            const size_t src = (((size_t)page * a.n_kv_heads + g) * kPageSize + slot) * a.head_dim + 8 * c;
            kv = *reinterpret_cast<const uint4 *>(a.k_pool + src);
            vv = *reinterpret_cast<const uint4 *>(a.v_pool + src);
        } else {
            atomicOr(a.err, kErrBadPage);
        }
        *reinterpret_cast<uint4 *>(a.k_out + dst) = kv;
        *reinterpret_cast<uint4 *>(a.v_out + dst) = vv;
    }
}

// grid (pages covering [from, len), Hkv): block copies the positions of one page of one KV head
// from the contiguous source into the pool's dense layout.
__global__ __launch_bounds__(256) void scatter_kernel(ScatterArgs a)
{
    const int g = blockIdx.y;
    const int pidx = a.from / kPageSize + blockIdx.x;
    const int page = a.page_row[pidx];
    if (page < 0 || page >= a.n_pool_pages) {
        if (threadIdx.x == 0 && a.err) atomicOr(a.err, kErrBadPage);
        return;
    }
    const int cpr = a.head_dim / 8;
    for (int i = threadIdx.x; i < kPageSize * cpr; i += blockDim.x) {
        const int slot = i / cpr, c = i % cpr, pos = pidx * kPageSize + slot;
        if (pos < a.from || pos >= a.len) continue;
        const size_t src = ((size_t)g * (a.len - a.from) + (pos - a.from)) * a.head_dim + 8 * c;
        const size_t dst = (((size_t)page * a.n_kv_heads + g) * kPageSize + slot) * a.head_dim + 8 * c;
        *reinterpret_cast<uint4 *>(a.k_pool + dst) = *reinterpret_cast<const uint4 *>(a.k_src + src);
        *reinterpret_cast<uint4 *>(a.v_pool + dst) = *reinterpret_cast<const uint4 *>(a.v_src + src);
    }
}

// Read-only streaming probe: block b reads the 16-byte words [b * chunk, (b + 1) * chunk) of the
// buffer, its threads interleaved, U loads in flight per thread, non-temporal like the K/V
// stream of the partial kernel; the words are folded into one value so the loads are kept.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int U>
__global__ void read_probe_kernel(const u32x4 *__restrict__ p, size_t n_vec, size_t chunk, uint32_t *sink)
{
    const size_t b0 = (size_t)blockIdx.x * chunk;
    const size_t e = b0 + chunk < n_vec ? b0 + chunk : n_vec;
    const size_t step = blockDim.x;
    uint32_t acc = 0;
    size_t i = b0 + threadIdx.x;
    for (; i + (U - 1) * step < e; i += U * step) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(p + i + u * step);
#pragma unroll
        for (int u = 0; u < U; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    for (; i < e; i += step) {
        const u32x4 v = __builtin_nontemporal_load(p + i);
        acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    if (acc == 0x9e3779b9u) sink[blockIdx.x % 64] = acc;  // practically never: keeps the loads alive
}

}  // namespace

hipError_t launch_read_probe(const void *buf, size_t bytes, int blocks, int threads, int unroll, uint32_t *sink,
                             hipStream_t s)
{
    const size_t n_vec = bytes / 16;
    const size_t chunk = (n_vec + blocks - 1) / blocks;
    const u32x4 *p = static_cast<const u32x4 *>(buf);
    switch (unroll) {
    case 4: read_probe_kernel<4><<<blocks, threads, 0, s>>>(p, n_vec, chunk, sink); break;
    case 8: read_probe_kernel<8><<<blocks, threads, 0, s>>>(p, n_vec, chunk, sink); break;
    case 16: read_probe_kernel<16><<<blocks, threads, 0, s>>>(p, n_vec, chunk, sink); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_scatter(const ScatterArgs &a, hipStream_t s)
{
    if (a.len <= a.from) return hipSuccess;
    const int blocks = (a.len + kPageSize - 1) / kPageSize - a.from / kPageSize;
    scatter_kernel<<<dim3(blocks, a.n_kv_heads), dim3(256), 0, s>>>(a);
    return hipGetLastError();
}

// Explicit-mode merges that take several rows per block: up to eight parts (one batch) at any size,
// and up to 32 from 2048 rows.  Measured (us, d 128, one block per row against several rows per
// block): 12800 rows 4 parts 12.7 / 4.5, 3200 rows 16 parts 5.6 / 4.2, 40 rows 8 parts 2.9 / 2.6; on
// the other side of the line 640 rows 16 parts 3.2 / 3.5, 1280 rows 64 parts 9.1 / 11.4, 40 rows 64
// parts 3.5 / 7.9, where a thread's batches follow one another.
bool several_rows_per_block(const MergeArgs &a)
{
    return !a.plan && (a.n_parts <= kMergeBatch || (a.n_parts <= 4 * kMergeBatch && a.rows >= 2048));
}

template <int HD>
void launch_merge_hd(const MergeArgs &a, hipStream_t s)
{
    const dim3 block(256);
    if (several_rows_per_block(a)) {
        const int per_block = 1024 / HD;
        merge_rows_kernel<HD><<<dim3((a.rows + per_block - 1) / per_block), block, 0, s>>>(a);
    } else if (!a.plan) {
        merge_kernel<HD, MergeParts::kExplicit, false><<<dim3(a.rows), block, 0, s>>>(a);
    } else {
        const dim3 rows(a.n_q_heads, a.rows / a.n_q_heads), step(rows.x + 1, rows.y);
        if (a.even_bpi > 0 && a.step_mode)
            merge_kernel<HD, MergeParts::kEven, true><<<step, block, 0, s>>>(a);
        else if (a.even_bpi > 0)
            merge_kernel<HD, MergeParts::kEven, false><<<rows, block, 0, s>>>(a);
        else if (a.step_mode)
            merge_kernel<HD, MergeParts::kPlan, true><<<step, block, 0, s>>>(a);
        else
            merge_kernel<HD, MergeParts::kPlan, false><<<rows, block, 0, s>>>(a);
    }
}

hipError_t launch_merge(const MergeArgs &a, int head_dim, hipStream_t s)
{
    if (a.rows <= 0) return hipSuccess;
    if (head_dim == 128)
        launch_merge_hd<128>(a, s);
    else if (head_dim == 64)
        launch_merge_hd<64>(a, s);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_append(const AppendArgs &a, int n_seqs, hipStream_t s)
{
    if (n_seqs <= 0) return hipSuccess;
    append_kernel<<<dim3(n_seqs), dim3(256), 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_gather(const GatherArgs &a, hipStream_t s)
{
    if (a.out_len <= a.begin) return hipSuccess;
    gather_kernel<<<dim3((a.out_len - a.begin + kPageSize - 1) / kPageSize, a.n_kv_heads), dim3(256), 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace fka
