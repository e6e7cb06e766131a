// Instruction prefill at the fork as a tiled multi-query attention kernel (gfx950, wave64).
//
// After a fork every branch b takes n instruction tokens at once (paper Sec. 3.3: the snapshot
// of the shared context followed by a short branch-specific instruction; Sec. 4.4: a branch's
// load is dominated by prefill over the cached prefix).  Token t of branch b is virtual sequence
// s = b n + t; its G query rows (one per query head of a KV head) attend to the whole shared
// prefix and to b's suffix positions [0, L_b + t] (causal within the instruction).  With N n G
// query rows per KV head sharing one prefix, this stage is a dense contraction: every prefix
// key is scored against hundreds of rows, so it runs on the matrix cores and is bound by their
// rate and by the vector work of the online softmax, not by HBM.
//
// Work: the rows of KV head g are cut into units of 32 consecutive rows (row i of the head is
// query head g G + i mod G of sequence i / G), one unit per wave.  A block of eight waves takes
// up to eight units of one KV head (the units spread evenly over the blocks of a range) over one
// range of key tiles (64 keys each); the keys are split into R ranges so that the blocks fill
// the device.  Each wave writes one normalised partial (o, lse) per row for its range, and
// the merge kernel combines a row's R partials (its explicit mode).
//   * K and V tiles go from HBM (or L2: the blocks of one KV head and range run on one XCD when
//     the KV heads are a multiple of 8 apart in the grid order) into LDS by DMA
//     (buffer_load_dwordx4 ... lds) into four tile buffers (two read while two load), each
//     tile loaded once by the block (every wave moves 8 of its 64 rows) and read by all eight
//     waves;
//   * the two waves of a SIMD alternate between matrix and vector work, in two phases per tile
//     with a block barrier between them: while one takes p.v of the previous tile and q.k of
//     this one (at raised priority), the other takes a softmax, and then the roles swap;
//   * S^T = K Q^T and O^T += V^T P^T run on v_mfma_f32_16x16x32_bf16 with keys on M, so each
//     lane owns two query rows of the online softmax (rows l16 and 16 + l16 of the unit) and
//     16 keys of each per tile; P enters the second product as two bf16 terms (hi + lo);
//   * K is read from LDS in the A-operand layout, V transposed with ds_read_b64_tr_b16, both
//     xor-swizzled by row so that a read touches every bank once, and both two groups of operands
//     ahead of the products;
//   * a row's reference of the exponentials moves only when its p have grown past a limit;
//   * the keys past the prefix's whole tiles -- its last Lp mod 64, then the suffix keys of every
//     branch the block's rows belong to -- form tiles of eight 8-key groups, each group of one branch,
//     which go through the same buffers; each row is masked to its own branch and causal limit.
//     The ranges share these tiles like the others (their number follows from the suffix lengths
//     on the device).  A non-finite value of a suffix is replaced by zero for the product and the rows
//     that read its key are made NaN, so that it reaches no row of another branch or of an earlier
//     token.
// What bounds it: beside a wave that issues matrix products at full rate the other wave of the SIMD
// gets one vector issue per 8.7 cycles (two per product), so a step cannot be shorter than 2 x 96
// products (3340 cycles) nor than the two softmaxes' ~225 issue slots each (3900); it takes 3940
// (32k prefix, 64 tokens x 5 branches, 40 / 8 heads), where the chip's power limit holds
// the clock at 2.2 of 2.4 GHz: 1.79 us, or 229 of the kernel's 260 us for the 128 tiles of a range (the rest: the start, the tail, the
// partials' stores at the end).  With the operands read in bursts that were waited for whole, a
// maximum per tile and the keys past the whole tiles read wave by wave, one round trip to memory per
// 32 keys (25000 cycles in the last range), it took 4920: 292 us a call against 265 now, 235
// against 211 at 256 tokens x 1 sequence over 33.8k keys, 74.5 against 65.5 at 16 x 5 over 23k.  (The sums
// of p as one more d tile of ones take 24 vector slots away and add 8 products: 277 us; the products' energy
// counts, not the slots.)
// A call of few keys per block is bound by its start and by whole steps of 1.5-2 us: the split's divisors
// come from the plan as exact products, the lengths are requested ahead of the tiles, and the
// ranges are cut for two steps where the partials stay small (1.2 us less of start, 1.7 us per step not
// taken: 320 rows 600 keys, 2 KV heads, 20.1 us against 14.9; 50 rows 2000 keys, 8 KV heads, 17.0 against 13.1).
#include <type_traits>
#include <utility>

#include "internal.h"
#include "scan64.h"

namespace fka {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(4))) const int32_t const_i32;

constexpr int KT = 64;             // keys per prefix tile
constexpr int NW = 8;              // waves per block (two per SIMD)
constexpr int STAGES = 4;          // prefix tile buffers: two read, two loading
constexpr int GRP = 8;             // keys per group of a tail tile (what one wave loads of a tile)
constexpr float kLn2 = 0.693147180559945309f;
constexpr float kRescaleLimit = 256.f;  // a lane's sum of a row's p over a tile past which the row's reference moves
constexpr float kNoKey = 3.402823466e38f;  // minus the reference of a row without keys: the largest float

static_assert(STAGES == 4, "the tile loop is unrolled over its four buffers");

__device__ inline f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ inline int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Raw buffer resource over [base, base + bytes), built from wave-uniform values.
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const char *base, int bytes)
{
    const uint64_t b = (uint64_t)base;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    const int n = __builtin_amdgcn_readfirstlane(bytes);
    return __builtin_amdgcn_make_buffer_rsrc((void *)(((uint64_t)hi << 32) | lo), 0, n, 0x00020000);
}

// 16 bytes per lane into LDS at dst + 16 * lane (LDS DMA), default cache policy: the other
// blocks of the KV head read the same tile from L2.  Kept outside the kernel template (used
// there directly, the builtin stops the host compiler from emitting the launch stub).
template <int OFFSET>
__device__ inline void dma16(__amdgpu_buffer_rsrc_t r, lds_void *dst, uint32_t voff)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, voff, 0, OFFSET, 0);
}

__device__ inline int32_t scalar_load(const int32_t *p) { return *(const_i32 *)p; }

template <int N>
__device__ inline void wait_vm()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

template <typename F, int... I>
__device__ inline void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ inline void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// max(a, b) in one instruction, for values that hold no signalling NaN (see max3 below).
__device__ inline float max2(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Maxima of two rows, x0 and x1, over lanes l, l ^ 16, l ^ 32, l ^ 48 (the four lanes holding a query
// row): the first exchange leaves row 0 in the lower half of the wave and row 1 in the upper, the
// last spreads both.  The inputs are maxima of matrix-core results (no signalling NaN).
__device__ inline void max_over_rows2(float &x0, float &x1)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
    const float x = max2(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = max2(__uint_as_float(b[0]), __uint_as_float(b[1]));
    const auto c = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    x0 = __uint_as_float(c[0]);
    x1 = __uint_as_float(c[1]);
}

__device__ inline float sum_over_rows(float x)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// LDS reads as inline assembly (the builtins make the compiler wait for every LDS DMA in
// flight, which would drain the tiles being prefetched); valid after lds_wait().
template <int OFFSET>
__device__ inline u32x4 ds_read_b128_at(uint32_t addr)
{
    static_assert(OFFSET >= 0 && OFFSET < 65536, "ds offset field");
    u32x4 r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "i"(OFFSET) : "memory");
    return r;
}

template <int OFFSET>
__device__ inline uint64_t ds_read_b64_at(uint32_t addr)
{
    static_assert(OFFSET >= 0 && OFFSET < 65536, "ds offset field");
    uint64_t r;
    asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "i"(OFFSET) : "memory");
    return r;
}

// ds_read_b64_tr_b16: within each group of 16 lanes, lane i receives element i % 4 of the rows
// addressed by lanes i / 4, 4 + i / 4, 8 + i / 4 and 12 + i / 4 (the transpose of a 16 x 4 block).
typedef long vtr_t;
template <int OFFSET>
__device__ inline vtr_t ds_read_tr16(uint32_t addr)
{
    static_assert(OFFSET >= 0 && OFFSET < 65536, "ds offset field");
    vtr_t r;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "i"(OFFSET) : "memory");
    return r;
}

__device__ inline void lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Waits until at most N LDS reads are outstanding.
template <int N>
__device__ inline void lds_wait_to()
{
    static_assert(N >= 0 && N < 16, "lgkmcnt range");
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"i"(N) : "memory");
}

// Every lane writes the same 8 bytes at one address (valid for the block after a barrier that waits for LDS).
__device__ inline void ds_write_b64(uint32_t addr, uint64_t x)
{
    asm volatile("ds_write_b64 %0, %1" ::"v"(addr), "v"(x) : "memory");
}

// Block barrier after this wave's LDS reads have returned (global loads stay in flight).
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Sixteen wait states between matrix-core ops and the first vector read of their results (the
// toolchain's own count for this op on gfx950 was seen to fall short in the decode kernel).
__device__ inline void xdl_result_wait()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7\n\ts_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// max(a, b, c) in one instruction.  fmaxf on a matrix-core result makes the compiler quiet a
// possible signalling NaN first (one more instruction per value); the matrix cores produce
// only quiet NaNs, which v_max3_f32 ignores as fmaxf does.
__device__ inline float max3(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Maximum of n values as a tree of v_max3_f32.
template <int N>
__device__ inline float max_of(const float (&v)[N])
{
    static_assert(N >= 3, "at least three values");
    if constexpr (N == 3) {
        return max3(v[0], v[1], v[2]);
    } else {
        constexpr int M = (N + 2) / 3;
        float w[M];
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const int k = 3 * i;
            w[i] = (k + 2 < N) ? max3(v[k], v[k + 1], v[k + 2]) : (k + 1 < N) ? max2(v[k], v[k + 1]) : v[k];
        }
        if constexpr (M < 3)
            return max2(w[0], w[M - 1]);
        else
            return max_of(w);
    }
}

__device__ inline int opaque_lane_id()
{
    int v;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(v));
    return v;
}

__device__ inline bf16x8 join_tr16(vtr_t lo, vtr_t hi)
{
    const s16x4 a = __builtin_bit_cast(s16x4, lo), b = __builtin_bit_cast(s16x4, hi);
    const short __attribute__((ext_vector_type(8))) v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    return __builtin_bit_cast(bf16x8, v);
}

// Splits p into hi + lo, both bf16 and both rounded to nearest: what is lost is 2^-18 of p.  (Cutting p off for
// hi takes as many instructions and loses twice that: 4.5e-6 of a result instead of 2.3e-6.)
// Packs the values of two key groups (four each) into the B operand of one p.v product.
// (v_dot2_f32_bf16 over the packed hi terms gives p - hi in one instruction instead of two, but
// measured 5% more cycles per tile.)
__device__ inline void split_p(const float (&p)[8], bf16x8 &hi, bf16x8 &lo)
{
    uint32_t hw[4];
    float r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) hi[i] = (__bf16)p[i];
    __builtin_memcpy(hw, &hi, sizeof(hw));
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = p[i] - __uint_as_float(i & 1 ? hw[i / 2] & 0xffff0000u : hw[i / 2] << 16);
#pragma unroll
    for (int i = 0; i < 8; ++i) lo[i] = (__bf16)r[i];
}

// A matrix phase works in groups of products: NV groups of p.v (two d tiles of a 32-key k-step: 8
// products, 128 cycles), then NK of q.k (one 16-key score tile: 8 products at d = 128), with VR or KR LDS
// reads each.  Operands are read two groups ahead (three groups in flight: the counter of LDS reads
// holds 15), so that only the first group waits for LDS, also while a tile's loads are being written there: reads return in order, so
// "at most N outstanding", N the reads of the groups requested behind it, means a group's are in.
template <int NV, int NK, int VR, int KR>
struct MatrixPlan {
    static constexpr int AHEAD = 2;
    static_assert((AHEAD + 1) * (VR > KR ? VR : KR) <= 15, "reads in flight");
    // the group before which group j is requested, in a phase that starts at group `first`
    static constexpr int due(int j, int first)
    {
        const int d = j - AHEAD;
        return d > first ? d : first;
    }
    static constexpr int behind(int q, int first)
    {
        int n = 0;
        for (int j = q + 1; j < NV + NK; ++j)
            if (due(j, first) <= q) n += j < NV ? VR : KR;
        return n;
    }
};

// The kernel's lambdas are inlined whatever their size: a call would keep what they capture in
// scratch memory.
#define INLINE __attribute__((always_inline))

// Layout of the 16x16x32 products: the output tile holds 16 keys (or 16 d) x 16 query rows; lane
// (q4, l16) = (l / 16, l mod 16) owns column l16 and rows 4 q4 + j (register j).  (The 32x32x16 op
// needs fewer cross-lane steps, but the same products take half as much energy again there: at the
// power limit, registers only, 1370 TFLOP/s against 2000; here the clock fell from 2.4 to 2.0 GHz
// and the call took as long.)
template <int HD, bool PAGED>
__device__ INLINE inline void prefill_tiles(const PrefillArgs &a)
{
    constexpr int ROWB = HD * 2;            // bytes per key row
    constexpr int CPR = HD / 8;             // 16-byte chunks per key row
    constexpr int NC = HD / 32;             // k-steps of the q.k product
    constexpr int NE = HD / 16;             // 16-wide d tiles of the output
    constexpr int MT = KT / 16;             // 16-key score tiles per prefix tile
    constexpr int KS = KT / 32;             // 32-key k-steps of p.v per prefix tile
    constexpr int EG = 2;                   // d tiles per group of V operands
    constexpr int KBYTES = KT * ROWB;       // K (or V) of one prefix tile
    constexpr int V_LDS = STAGES * KBYTES;  // K buffers first, then V buffers
    constexpr int LDS_BYTES = 2 * STAGES * KBYTES;
    constexpr int RPI = 64 / CPR;           // key rows one DMA instruction moves
    constexpr int DMAS = 8 / RPI;           // DMA instructions for a wave's 8 rows of K (or V)
    static_assert(NW * GRP == KT, "one group of a tile per wave");
    static_assert((STAGES - 1) * KBYTES + (KT - 16) * ROWB < 65536, "LDS offsets fit the immediate field");
    // LDS chunk position of chunk c of row r: c ^ swz(r).  K is read 16 consecutive rows at one
    // chunk (ds_read_b128), V 8 consecutive rows at 2 consecutive chunks (the transposed read, half
    // a wave): both then touch every 16-byte slot of the 256-byte bank line once.
    auto swz_k = [](int r) { return CPR == 16 ? (r & 15) : ((r >> 1) & 7); };
    auto swz_v = [](int r) { return CPR == 16 ? 2 * (r & 7) : 2 * ((r >> 1) & 3); };

    __shared__ __attribute__((aligned(1024))) char lds[LDS_BYTES];
    // per tile buffer, the groups of a tail tile: branch and last key (see issue_tail)
    __shared__ __attribute__((aligned(16))) int2 s_grp[STAGES][NW];

    const int tid = threadIdx.x;
    const int lane = tid & 63, l16 = lane & 15, q4 = lane >> 4;
    const int wave = uni(tid >> 6);
    const int Hkv = a.n_kv_heads, G = a.group, Hq = a.n_q_heads;
    const int n = a.n_tokens, N = a.n_branches;
    const int S = N * n, rows_head = S * G;
    const int Lp = a.prefix_len;

    // block -> (KV head, unit group, range); the KV head varies fastest so that with Hkv a
    // multiple of 8 a head's blocks all land on one XCD (block b runs on XCD b mod 8)
    const int vb = blockIdx.x;
    const int rest = vb / a.split.kv_heads, g = vb - rest * Hkv;
    const int r = rest / a.split.unit_groups, ug = rest - r * a.unit_groups;
    // the units spread evenly over the groups (at most eight each): blocks of one range then
    // stream its tiles at the same pace, so each tile is fetched once into the XCD's L2 for all
    const int unit_a = ug * a.split.units_each + min(ug, a.split.units_more);
    const int unit_z = unit_a + a.split.units_each + (ug < a.split.units_more ? 1 : 0);
    const int u = unit_a + wave;
    const bool active = u < unit_z;
    const int R = a.ranges, RP = a.prefix_ranges;
    const int PT = a.prefix_tiles;

    // ---- the block's keys: the prefix's whole tiles, then the tail -- the prefix's last Lp mod 64 keys
    // (every row reads them) and the suffix keys of the branches its rows belong to, each branch up
    // to the last key any of the block's rows reads -- in groups of eight keys, eight groups to a tile.
    // The first RP ranges share the prefix: range r takes its tiles [s0, s0 + nmain) (known from the plan,
    // so their loads do not wait for the suffix lengths).  All R take tail tiles, as below.
    const int pre_each = a.split.pre_each, pre_more = a.split.pre_more;
    const int s0 = r * pre_each + min(r, pre_more), nmain = r < RP ? pre_each + (r < pre_more ? 1 : 0) : 0;

    const int row_z = min(rows_head, unit_z * 32);
    const int br_a = (unit_a * 32) / a.split.branch_rows;
    const int seq_z = (row_z - 1) / a.split.group, br_z = (row_z - 1) / a.split.branch_rows;
    const int tail0 = PT * KT, pre_groups = (Lp - tail0 + GRP - 1) / GRP;
    // Lane i of a chunk of 64 branches: branch br_first + i's length before the instruction, and the
    // inclusive scan of the branches' groups (br_base groups precede the chunk)
    int br_len = 0, br_scan = 0, br_first = br_a, br_base = pre_groups, n_groups = 0;
    auto request_branches = [&](int first) INLINE { return first + lane <= br_z ? a.suffix_len[first + lane] : 0; };
    auto take_branches = [&](int first, int raw) INLINE {
        const int b = first + lane;
        br_len = min(max(raw, 0), a.max_suffix_len - n);
        if (b <= br_z && br_len != raw) atomicOr(a.err, kErrSuffixClamped);
        br_scan = scan64(b <= br_z ? (br_len + min(n - 1, seq_z - b * n) + GRP) / GRP : 0);  // (keys + 7) / 8, keys = len + t + 1
        br_first = first;
    };
    // (requested in front of the first tile: loads return in order)
    const int raw_a = request_branches(br_a);

    // DMA: this wave moves tile rows [8 wave, 8 wave + 8): instruction ii writes rows
    // 8 wave + RPI ii + lane / CPR, lane's LDS chunk position lane % CPR, which holds the row's
    // global chunk position ^ swizzle(row)
    uint32_t koff[DMAS], voff[DMAS];
#pragma unroll
    for (int ii = 0; ii < DMAS; ++ii) {
        const int tl = RPI * ii + lane / CPR, pos = lane % CPR, T = 8 * wave + tl;
        koff[ii] = tl * ROWB + 16 * (pos ^ swz_k(T));
        voff[ii] = tl * ROWB + 16 * (pos ^ swz_v(T));
    }
    // ---- prefix tile loads: this wave's 8 rows of tile `tile` into stage `st`
    bool bad_page = false;
    const char *const pk = reinterpret_cast<const char *>(PAGED ? a.k_pool : a.prefix_k);
    const char *const pv = reinterpret_cast<const char *>(PAGED ? a.v_pool : a.prefix_v);
    // paged: lane i holds the page id of this wave's rows of tile page_base + i (a scalar load per tile
    // would put its latency into every step); prefix pages have the same ids in every branch's row
    // (branch 0's is read)
    int32_t page_ids = 0;
    int page_base = s0;
    auto request_pages = [&](int tile) INLINE {
        page_base = tile;
        const int i = (int)min((int64_t)(tile + lane) * (KT / kPageSize) + wave * 8 / kPageSize, (int64_t)a.max_pages - 1);
        page_ids = a.page_table[i];
        asm volatile("" : "+v"(page_ids));  // waited for here: a wait at each use would drain the tiles in flight
    };
    if constexpr (PAGED) request_pages(s0);
    // `bytes` bytes of K and V rows into this wave's eight rows of stage st
    auto load_rows = [&](const char *ksrc, const char *vsrc, int bytes, int st) INLINE {
        const __amdgpu_buffer_rsrc_t rk = make_rsrc(ksrc, bytes), rv = make_rsrc(vsrc, bytes);
        char *kd = &lds[st * KBYTES + 8 * wave * ROWB];
        char *vd = &lds[V_LDS + st * KBYTES + 8 * wave * ROWB];
#pragma unroll
        for (int ii = 0; ii < DMAS; ++ii)
            dma16<0>(rk, (lds_void *)(__attribute__((address_space(3))) char *)(kd + ii * RPI * ROWB), koff[ii]);
#pragma unroll
        for (int ii = 0; ii < DMAS; ++ii)
            dma16<0>(rv, (lds_void *)(__attribute__((address_space(3))) char *)(vd + ii * RPI * ROWB), voff[ii]);
    };
    // this wave's rows of a whole tile (without branches and in few scalar steps: they stand in every
    // step of the inner loop)
    const uint64_t page_bytes = (uint64_t)Hkv * kPageSize * ROWB;
    const size_t wave_off = PAGED ? (size_t)g * kPageSize * ROWB + (8 * wave % kPageSize) * ROWB
                                  : ((size_t)g * Lp + 8 * wave) * ROWB;
    const char *const pkw = pk + wave_off, *const pvw = pv + wave_off;
    auto issue_prefix = [&](int tile, int st) INLINE {
        if constexpr (PAGED) {
            const uint32_t page = (uint32_t)__builtin_amdgcn_readlane(page_ids, tile - page_base);
            const bool bad = page >= (uint32_t)a.n_pool_pages;
            bad_page |= bad;
            const uint64_t off = page * page_bytes;
            load_rows(bad ? pk : pkw + off, bad ? pv : pvw + off, bad ? 0 : 8 * ROWB, st);
        } else {
            const uint64_t off = (uint64_t)(uint32_t)tile * (KT * ROWB);
            load_rows(pkw + off, pvw + off, 8 * ROWB, st);
        }
    };
    // the first tiles' loads go ahead of everything that they do not need
    if (nmain > 0) issue_prefix(s0, 0);

    // ---- query rows (B operand of S^T): lane holds unit row 16 t + l16, d = 32 c + 8 q4 .. +7
    bf16x8 qb[2][NC];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int lr = u * 32 + 16 * t + l16;
#pragma unroll
        for (int c = 0; c < NC; ++c) qb[t][c] = bf16x8{};
        if (active && lr < rows_head) {
            const int s = lr / a.split.group, h = g * G + lr - s * G;
            const uint16_t *qp = a.q + ((size_t)s * Hq + h) * HD + 8 * q4;
#pragma unroll
            for (int c = 0; c < NC; ++c) qb[t][c] = *reinterpret_cast<const bf16x8 *>(qp + 32 * c);
        }
    }

    if (nmain > 1) issue_prefix(s0 + 1, 1);

    // ---- per-lane constants
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)&lds[0];
    // K A-operand reads: row 16 i + l16 (i = M tile, an immediate), chunk 4 c + q4
    uint32_t kaddr[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) kaddr[c] = lds0 + l16 * ROWB + 16 * ((4 * c + q4) ^ swz_k(l16));
    // V^T reads (transposed): lane (q4, l16) addresses row 4 q4 + l16 / 4, d = 16 e + 4 (l16 % 4); rows
    // 16 m further are an immediate away with the same swizzle
    uint32_t vaddr[NE];
    {
        const int m4 = l16 & 3, T = 4 * q4 + (l16 >> 2);
#pragma unroll
        for (int e = 0; e < NE; ++e)
            vaddr[e] = lds0 + V_LDS + T * ROWB + 16 * ((2 * e + (m4 >> 1)) ^ swz_v(T)) + (m4 & 1) * 8;
    }

    // Tail tile j: this wave loads group 8 j + wave of the tail and leaves the group's branch (-1: the
    // prefix, -2: no group) and limit in s_grp: a row of the branch with token t reads the group's
    // keys k <= limit + t, every row those of the prefix with k <= limit.
    auto issue_tail = [&](int j, int st) INLINE {
        const int idx = j * NW + wave;
        int b = -2, limit = -1, rows_ok = 0, pos = 0;
        if (idx < pre_groups) {
            b = -1;
            pos = GRP * idx;
            limit = Lp - tail0 - 1 - pos;
            rows_ok = min(GRP, limit + 1);
        } else if (idx < n_groups &&
                   find_chunk(idx, br_z, br_first, br_base, [&]() INLINE { return __builtin_amdgcn_readlane(br_scan, 63); },
                              [&](int first) INLINE { take_branches(first, request_branches(first)); })) {
            const int k = idx - br_base;
            const int i = uni(__builtin_ctzll(__builtin_amdgcn_ballot_w64(br_scan > k)));
            b = br_first + i;
            const int L = __builtin_amdgcn_readlane(br_len, i);
            const int keys = L + min(n - 1, seq_z - b * n) + 1;
            pos = GRP * (k - (__builtin_amdgcn_readlane(br_scan, i) - (keys + GRP - 1) / GRP));
            limit = L - pos;
            rows_ok = min(GRP, keys - pos);
        } else if (idx < n_groups && lane == 0) {
            atomicOr(a.err, kErrBadSchedule);  // the lengths shrank while the kernel read them: the group is left out
        }
        size_t off = 0;
        if (rows_ok > 0) {
            if constexpr (PAGED) {
                const int at = b < 0 ? (tail0 + pos) / kPageSize : (Lp + kPageSize - 1) / kPageSize + pos / kPageSize;
                const int32_t page = scalar_load(a.page_table + (size_t)max(b, 0) * a.max_pages + uni(min(at, a.max_pages - 1)));
                const bool bad = page < 0 || page >= a.n_pool_pages;
                bad_page |= bad;
                rows_ok = bad ? 0 : rows_ok;
                off = bad ? 0 : (((size_t)page * Hkv + g) * kPageSize + pos % kPageSize) * ROWB;
            } else {
                off = (b < 0 ? (size_t)g * Lp + tail0 + pos : ((size_t)b * Hkv + g) * a.suffix_cap + pos) * ROWB;
            }
        }
        const bool pre = b < 0 || PAGED;
        load_rows((pre ? pk : reinterpret_cast<const char *>(a.suffix_k)) + off,
                  (pre ? pv : reinterpret_cast<const char *>(a.suffix_v)) + off, rows_ok * ROWB, st);
        ds_write_b64((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)&s_grp[st][wave],
                     (uint64_t)(uint32_t)b | ((uint64_t)(uint32_t)limit << 32));
    };
    // the range's share of the tail, now that the lengths are needed
    take_branches(br_a, raw_a);
    n_groups = pre_groups + __builtin_amdgcn_readlane(br_scan, 63);
    if (br_z - br_a >= 64) {  // more branches than lanes: count the rest, then back to the first chunk
        for (int first = br_a + 64; first <= br_z; first += 64) {
            take_branches(first, request_branches(first));
            n_groups += __builtin_amdgcn_readlane(br_scan, 63);
        }
        take_branches(br_a, request_branches(br_a));
    }
    int tail_t0, tail_n;
    tail_share(a.split, RP, R, (n_groups + NW - 1) / NW, r, tail_t0, tail_n);
    const int ntot = nmain + tail_n;
    // paged: the page ids of the next n tiles from the range's tile i are in page_ids
    auto have_pages = [&](int i, int n) INLINE {
        if constexpr (PAGED)
            if (s0 + i + n - page_base > 64) request_pages(s0 + i);
    };
    auto issue = [&](int i) INLINE {  // the range's tile i into buffer i mod 4
        if (i < nmain) {
            have_pages(i, 1);
            issue_prefix(s0 + i, i % STAGES);
        } else
            issue_tail(tail_t0 + i - nmain, i % STAGES);
    };

    // ---- online softmax state: lane owns unit rows l16 (t = 0) and 16 + l16 (t = 1).  nm is minus
    // the row's reference in log2 units, the maximum of the scores that last moved it: p = 2^(score -
    // reference), sums and accumulator are relative to it.  The lowest number before the row's first
    // key: p of a key is then past every limit and p of a masked one 0.
    f32x4 acc[2][NE];
    float nm[2] = {kNoKey, kNoKey}, l_run[2] = {0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < NE; ++e) acc[t][e] = f32x4{0.f, 0.f, 0.f, 0.f};

    // p of a tile's scores (x[t][4 i + j]: key 16 i + 4 q4 + j, raw q.k or -inf) against the references
    // r as two bf16 terms per k-step of 32 keys, and this lane's sum of p per row.
    auto exps = [&](const float (&x)[2][4 * MT], const float (&r)[2], bf16x8 (&ph)[2][KS], bf16x8 (&pl)[2][KS],
                    float (&sum)[2]) INLINE {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            float ps[4];
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) {
                float p[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    p[j] = fast_exp2(__builtin_fmaf(x[t][8 * kk + j], a.scale_log2, r[t]));
                    ps[j & 3] = (kk == 0 && j < 4) ? p[j] : ps[j & 3] + p[j];
                }
                split_p(p, ph[t][kk], pl[t][kk]);
            }
            sum[t] = (ps[0] + ps[1]) + (ps[2] + ps[3]);
        }
    };
    // The references of the rows whose sum is past the limit in any of their four lanes moved to the tile's
    // maxima, sums and accumulator rescaled.  The other rows of the unit are left as they are, alpha 1 and
    // the same p, so that a row's bits do not depend on what the rows beside it hold.
    auto move_reference = [&](const float (&x)[2][4 * MT], const float (&sum)[2]) INLINE {
        float mx[2] = {max_of(x[0]), max_of(x[1])};
        max_over_rows2(mx[0], mx[1]);
        xdl_result_wait();
        const int row = opaque_lane_id() & 15;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            uint64_t over = __builtin_amdgcn_ballot_w64(sum[t] > kRescaleLimit);
            over |= over >> 32;
            over |= over >> 16;
            const float m_new = mx[t] * a.scale_log2;  // the scale is positive: the order is kept
            const bool move = ((uint32_t)over >> row & 1) != 0 && m_new > -nm[t];
            const float alpha = move ? fast_exp2(-nm[t] - m_new) : 1.f;  // 0 for a row's first keys
            l_run[t] *= alpha;
#pragma unroll
            for (int e = 0; e < NE; ++e) acc[t][e] *= alpha;
            nm[t] = move ? -m_new : nm[t];
        }
    };
    // A tile's softmax.  Any reference gives the same result while nothing overflows (all that it
    // scales is in fp32), so p is taken against the old one and only a row whose sum in a lane is past
    // kRescaleLimit leads to the path with the maxima: a maximum per tile costs 26 of 250 vector issue
    // slots, and beside a matrix wave those bound the step.  (A NaN row stays on the path without: the
    // larger of two sums, one of them NaN, is the other.)
    // `first`: the range's first tile, where every row with a key takes its reference.
    auto softmax = [&](const float (&x)[2][4 * MT], bf16x8 (&ph)[2][KS], bf16x8 (&pl)[2][KS], bool first) INLINE {
        float sum[2] = {INFINITY, INFINITY};
        if (!first) exps(x, nm, ph, pl, sum);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(fmaxf(sum[0], sum[1]) > kRescaleLimit) != 0, 0)) {
            move_reference(x, sum);
            exps(x, nm, ph, pl, sum);
        }
        l_run[0] += sum[0];
        l_run[1] += sum[1];
    };

    // p.v of EG d tiles from e0 and one k-step (32 keys: 4 q4 + j and 16 + 4 q4 + j)
    auto pv_mfma = [&](auto E0c, const vtr_t (&v)[EG][2], const bf16x8 (&ph)[2], const bf16x8 (&pl)[2]) INLINE {
        constexpr int e0 = decltype(E0c)::value;
#pragma unroll
        for (int e = 0; e < EG; ++e) {
            const bf16x8 va = join_tr16(v[e][0], v[e][1]);
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[t][e0 + e] = mfma16(va, ph[t], acc[t][e0 + e]);
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[t][e0 + e] = mfma16(va, pl[t], acc[t][e0 + e]);
        }
    };

    // ---- the range's tiles, two loading ahead, in two phases per tile.  The two
    // waves of a SIMD alternate between matrix and vector work: in phase 1 of step i the first
    // wave (waves 0..3) takes p.v of tile i - 1 and q.k of tile i while the second (waves 4..7)
    // takes the softmax of tile i - 1; in phase 2 the first takes the softmax of tile i while the
    // second takes p.v of tile i - 1 and q.k of tile i (p.v first, so that p and the new scores
    // are not live together).  A block barrier separates the phases; the
    // wave in its matrix phase runs at raised priority.  Four tile buffers: tiles i - 1 and i are
    // read during step i while i + 1 and i + 2 load.
    //
    constexpr int NG = KS * (NE / EG);  // groups of V operands per tile
    using plan = MatrixPlan<NG, MT, 2 * EG, NC>;
    auto read_v = [&](auto SOc, auto Gc, uint32_t dyn, vtr_t (&v)[EG][2]) INLINE {
        constexpr int kk = decltype(Gc)::value / (NE / EG), e0 = decltype(Gc)::value % (NE / EG) * EG;
        constexpr int o = decltype(SOc)::value + kk * 32 * ROWB;
#pragma unroll
        for (int e = 0; e < EG; ++e) {
            v[e][0] = ds_read_tr16<o>(vaddr[e0 + e] + dyn);
            v[e][1] = ds_read_tr16<o + 16 * ROWB>(vaddr[e0 + e] + dyn);
        }
    };
    auto read_k = [&](auto SOc, auto Mc, uint32_t dyn, bf16x8 (&k)[NC]) INLINE {
        constexpr int o = decltype(SOc)::value + decltype(Mc)::value * 16 * ROWB;
#pragma unroll
        for (int c = 0; c < NC; ++c) k[c] = __builtin_bit_cast(bf16x8, ds_read_b128_at<o>(kaddr[c] + dyn));
    };
    auto tie_v = [&](vtr_t (&v)[EG][2]) INLINE {
#pragma unroll
        for (int e = 0; e < EG; ++e) asm volatile("" : "+v"(v[e][0]), "+v"(v[e][1]));
    };
    auto tie_k = [&](bf16x8 (&k)[NC]) INLINE {
#pragma unroll
        for (int c = 0; c < NC; ++c) asm volatile("" : "+v"(k[c]));
    };
    auto qk_group = [&](auto Mc, const bf16x8 (&k)[NC], f32x4 (&sc)[2][MT]) INLINE {
        constexpr int mi = decltype(Mc)::value;
        sc[0][mi] = sc[1][mi] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int t = 0; t < 2; ++t) sc[t][mi] = mfma16(k[c], qb[t][c], sc[t][mi]);
    };
    // p.v of the tile at buffer offset SOP + dynp (PV) and q.k of the one at SO + dyn.
    auto matrix = [&](auto PVc, auto SOc, auto SOPc, uint32_t dyn, uint32_t dynp, f32x4 (&sc)[2][MT], const bf16x8 (&ph)[2][KS],
                      const bf16x8 (&pl)[2][KS]) INLINE {
        constexpr int first = decltype(PVc)::value ? 0 : NG, last = NG + MT;  // groups: V 0..NG-1, K NG..NG+MT-1
        constexpr int SETS = plan::AHEAD + 1;
        vtr_t v[SETS][EG][2];
        bf16x8 k[SETS][NC];
        auto request = [&](auto Jc) INLINE {
            constexpr int j = decltype(Jc)::value;
            if constexpr (j < NG)
                read_v(SOPc, Jc, dynp, v[j % SETS]);
            else
                read_k(SOc, std::integral_constant<int, j - NG>{}, dyn, k[(j - NG) % SETS]);
        };
        static_for<last - first>([&](auto Ic) INLINE {
            constexpr int q = first + decltype(Ic)::value;
            static_for<last - first>([&](auto Jc) INLINE {
                constexpr int j = first + decltype(Jc)::value;
                if constexpr (plan::due(j, first) == q) request(std::integral_constant<int, j>{});
            });
            lds_wait_to<plan::behind(q, first)>();
            if constexpr (q < NG)
                tie_v(v[q % SETS]);
            else
                tie_k(k[(q - NG) % SETS]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (q < NG) {
                constexpr int kk = q / (NE / EG);
                const bf16x8 h2[2] = {ph[0][kk], ph[1][kk]}, l2[2] = {pl[0][kk], pl[1][kk]};
                pv_mfma(std::integral_constant<int, q % (NE / EG) * EG>{}, v[q % SETS], h2, l2);
            } else {
                qk_group(std::integral_constant<int, q - NG>{}, k[(q - NG) % SETS], sc);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // (every tile of the inner loop is whole: no key mask, which would make the compiler copy the
    // scores into the masked path's registers)
    auto sm = [&](const f32x4 (&sc)[2][MT], bf16x8 (&ph)[2][KS], bf16x8 (&pl)[2][KS], auto &&also) INLINE {
        xdl_result_wait();
        also();
        float x[2][4 * MT];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 4 * MT; ++i) x[t][i] = sc[t][i >> 2][i & 3];
        softmax(x, ph, pl, false);
    };
    f32x4 sc[2][MT];
    bf16x8 ph[2][KS], pl[2][KS];
    using zero = std::integral_constant<int, 0>;
    // Step i of the inner loop, tile i in buffer B = i mod 4: q.k of tile i, p.v of tile i - 1 and the
    // load of tile i + 2, all whole prefix tiles.  The two roles run in loops of their own (a role
    // test in each phase would keep both roles' values live at once); both pass the same barriers.
    auto step = [&](int i, auto Bc, auto LEADc) INLINE {
        constexpr int B = decltype(Bc)::value;
        constexpr bool LEAD = decltype(LEADc)::value;
        using so_t = std::integral_constant<int, B * KBYTES>;
        using sop_t = std::integral_constant<int, ((B + STAGES - 1) % STAGES) * KBYTES>;
        auto mat = [&]() INLINE {
            __builtin_amdgcn_s_setprio(1);
            matrix(std::true_type{}, so_t{}, sop_t{}, 0u, 0u, sc, ph, pl);
            __builtin_amdgcn_s_setprio(0);
        };
        // the load of tile i + 2, among the softmax's vector work: in front of a matrix phase its scalar
        // work would hold up the products
        auto load = [&]() INLINE { issue_prefix(s0 + i + 2, (B + 2) % STAGES); };
        auto vec = [&]() INLINE {
            if (active)
                sm(sc, ph, pl, load);
            else
                load();
        };
        wait_vm<2 * DMAS>();
        lds_barrier();  // tile i is in LDS; every wave is done with tile i - 2
        if constexpr (LEAD) {
            if (active) mat();
        } else {
            vec();
        }
        lds_barrier();
        if constexpr (LEAD)
            vec();
        else if (active)
            mat();
    };

    // ---- the same step for any tile: the first (no p.v), the last (only p.v) and those of the tail,
    // where a wave skips a tile none of its rows reads (use) and masks the keys of each group past
    // each row's limit.  What follows describes the tile whose q.k was last taken.
    // A lane's four keys of score tile i are keys 4 (q4 mod 2) + j of group 2 i + q4 / 2.
    bool use = true, tail = false;
    int lim[2][MT];  // row t reads the keys k <= lim[t][i] of group 2 i + q4 / 2
    uint32_t suffix_groups = 0;  // bit i: that group holds suffix keys (not the prefix's, which every row reads)
#pragma unroll
    for (int i = 0; i < MT; ++i) lim[0][i] = lim[1][i] = KT;
    int row_bt[2];  // the rows' branch (past every branch beyond the head's rows) << 16 | token
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int lr = u * 32 + 16 * t + l16;
        const int br = lr / a.split.branch_rows;
        row_bt[t] = lr < rows_head ? br << 16 | (lr / a.split.group - br * n) : 0x7fff0000;
    }
    const uint32_t grp0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)&s_grp[0][0] + 8 * (q4 >> 1);
    auto any_qk = [&](int i) INLINE {
        use = true;
        tail = i >= nmain;
        if (!tail) {
#pragma unroll
            for (int q = 0; q < MT; ++q) lim[0][q] = lim[1][q] = KT;
        } else {
            uint64_t d[MT];
            static_for<MT>([&](auto Qc) INLINE {
                constexpr int q = decltype(Qc)::value;
                d[q] = ds_read_b64_at<16 * q>(grp0 + (i % STAGES) * (uint32_t)sizeof(s_grp[0]));
            });
            lds_wait();
#pragma unroll
            for (int q = 0; q < MT; ++q) asm volatile("" : "+v"(d[q]));
            int most = -1;
            suffix_groups = 0;
#pragma unroll
            for (int q = 0; q < MT; ++q) {
                const int b = (int)(uint32_t)d[q], base = (int)(d[q] >> 32);
                suffix_groups |= b >= 0 ? 1u << q : 0;
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    lim[t][q] = b == -1 ? base : b == row_bt[t] >> 16 ? base + (row_bt[t] & 0xffff) : -1;
                    most = max(most, lim[t][q]);
                }
            }
            use = __builtin_amdgcn_ballot_w64(most >= 0) != 0;
        }
        if (use) matrix(std::false_type{}, zero{}, zero{}, (uint32_t)(i % STAGES) * KBYTES, 0u, sc, ph, pl);
    };
    auto any_sm = [&](int i) INLINE {
        if (!use) return;
        xdl_result_wait();
        float x[2][4 * MT];
        const int k0 = 4 * ((opaque_lane_id() >> 4) & 1);  // the lane's first key of its groups
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 4 * MT; ++i)
                x[t][i] = (k0 + (i & 3) <= lim[t][i >> 2]) ? sc[t][i >> 2][i & 3] : -INFINITY;
        softmax(x, ph, pl, i == 0);
    };
    auto any_pv = [&](int i) INLINE {
        if (!use) return;
        const uint32_t dyn = (uint32_t)(i % STAGES) * KBYTES;
        constexpr int PG = NE < 4 ? NE : 4, GS = PG / EG;  // d tiles per round of reads
        static_for<KS * (NE / PG)>([&](auto Rc) INLINE {
            constexpr int kk = decltype(Rc)::value / (NE / PG), q0 = decltype(Rc)::value * GS;
            vtr_t v[GS][EG][2];
            static_for<GS>([&](auto Gc) INLINE {
                read_v(zero{}, std::integral_constant<int, q0 + decltype(Gc)::value>{}, dyn, v[decltype(Gc)::value]);
            });
            lds_wait();
            static_for<GS>([&](auto Gc) INLINE { tie_v(v[decltype(Gc)::value]); });
            if (tail) {
                // A non-finite value of a suffix group is zeroed for the product and the rows that read its
                // key are made NaN (through their sums), so that it reaches no row of another branch or of
                // an earlier token (a masked row's p is 0, and 0 times such a value would be NaN).  The
                // prefix's keys are read by every row: theirs stay in the product, as in the whole tiles.
                uint32_t bits = 0;
#pragma unroll
                for (int e = 0; e < PG; ++e)
#pragma unroll
                    for (int y = 0; y < 2; ++y) {
                        const uint64_t w = (uint64_t)v[e / EG][e % EG][y];
                        bits |= (((uint32_t)w & 0x7f807f80u) + 0x00800080u) |
                                ((((uint32_t)(w >> 32)) & 0x7f807f80u) + 0x00800080u);
                    }
                if (__builtin_expect(__builtin_amdgcn_ballot_w64((bits & 0x80008000u) != 0) != 0, 0)) {
                    // read y holds keys k0 + k (k = 0..3) of group 2 (2 kk + y) + q4 / 2, a half wave's group
                    const int k0 = 4 * ((opaque_lane_id() >> 4) & 1);
#pragma unroll
                    for (int y = 0; y < 2; ++y) {
                        // the exponent bits that count as non-finite (none for the prefix's keys)
                        const uint32_t bad = (suffix_groups >> (2 * kk + y) & 1) ? 0x7f80u : ~0u;
                        int first = 0x7fffffff;
#pragma unroll
                        for (int e = 0; e < PG; ++e) {
                            uint64_t w = (uint64_t)v[e / EG][e % EG][y];
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                if (((uint32_t)(w >> (16 * k)) & 0x7f80u) == bad) {
                                    first = min(first, k0 + k);
                                    w &= ~((uint64_t)0xffffu << (16 * k));
                                }
                            v[e / EG][e % EG][y] = (vtr_t)w;
                        }
#pragma unroll
                        for (int off = 1; off < 32; off <<= 1) first = min(first, __shfl_xor(first, off));
#pragma unroll
                        for (int t = 0; t < 2; ++t)
                            l_run[t] = lim[t][2 * kk + y] >= first ? __builtin_nanf("") : l_run[t];
                    }
                }
            }
            const bf16x8 h2[2] = {ph[0][kk], ph[1][kk]}, l2[2] = {pl[0][kk], pl[1][kk]};
            static_for<GS>([&](auto Gc) INLINE {
                constexpr int q = q0 + decltype(Gc)::value;
                pv_mfma(std::integral_constant<int, q % (NE / EG) * EG>{}, v[decltype(Gc)::value], h2, l2);
            });
        });
    };
    auto any_step = [&](int i, auto LEADc) INLINE {
        constexpr bool LEAD = decltype(LEADc)::value;
        auto mat = [&]() INLINE {
            __builtin_amdgcn_s_setprio(1);
            if (i > 0) any_pv(i - 1);
            if (i < ntot) any_qk(i);
            __builtin_amdgcn_s_setprio(0);
        };
        if (i + 1 < ntot)
            wait_vm<2 * DMAS>();
        else
            wait_vm<0>();
        lds_barrier();
        if (i + 2 < ntot) issue(i + 2);
        if (active) {
            if constexpr (LEAD)
                mat();
            else if (i > 0)
                any_sm(i - 1);
        }
        lds_barrier();
        if (active) {
            if constexpr (!LEAD)
                mat();
            else if (i < ntot)
                any_sm(i);
        }
    };
    // Step i between two whole tiles, with the buffers' offsets known at run time: what the unrolled
    // steps leave over, and ranges too short for them (the general step instead costs 0.3-0.5 us more each:
    // 5-7 tiles a block, 29.2 us against 27.8 at 320 rows 32k keys, 1 KV head).
    auto whole_step = [&](int i, auto LEADc) INLINE {
        constexpr bool LEAD = decltype(LEADc)::value;
        auto mat = [&]() INLINE {
            __builtin_amdgcn_s_setprio(1);
            matrix(std::true_type{}, zero{}, zero{}, (uint32_t)(i % STAGES) * KBYTES, (uint32_t)((i + STAGES - 1) % STAGES) * KBYTES, sc,
                   ph, pl);
            __builtin_amdgcn_s_setprio(0);
        };
        auto nothing = [&]() INLINE {};
        if (i + 1 < ntot)
            wait_vm<2 * DMAS>();
        else
            wait_vm<0>();
        lds_barrier();
        if (i + 2 < ntot) issue(i + 2);
        if (active) {
            if constexpr (LEAD)
                mat();
            else
                sm(sc, ph, pl, nothing);
        }
        lds_barrier();
        if (active) {
            if constexpr (LEAD)
                sm(sc, ph, pl, nothing);
            else
                mat();
        }
    };
    auto run = [&](auto LEADc) INLINE {
        any_step(0, LEADc);
        int i = 1;
        for (; i + 5 < nmain; i += STAGES) {  // (exits within the four steps made the compiler spill)
            have_pages(i + 2, STAGES);
            step(i, std::integral_constant<int, 1>{}, LEADc);
            step(i + 1, std::integral_constant<int, 2>{}, LEADc);
            step(i + 2, std::integral_constant<int, 3>{}, LEADc);
            step(i + 3, std::integral_constant<int, 0>{}, LEADc);
        }
        for (; i < nmain; ++i) whole_step(i, LEADc);
        for (; i <= ntot; ++i) any_step(i, LEADc);
    };
    if (ntot > 0) {
        if (nmain < 1) issue(0);
        if (nmain < 2 && ntot > 1) issue(1);
        if (wave < 4)
            run(std::true_type{});
        else
            run(std::false_type{});
    }
    if (PAGED && __builtin_amdgcn_ballot_w64(bad_page) != 0 && lane == 0) atomicOr(a.err, kErrBadPage);

    // ---- one normalised partial per row of the unit for range r
    if (!active) return;
    const int lane_c = opaque_lane_id();
    const int l16c = lane_c & 15, q4c = lane_c >> 4;
    const size_t rows_total = (size_t)S * Hq;
    xdl_result_wait();
    // An infinite value of the prefix meets hi and lo of p one after the other, and lo has either sign: inf - inf
    // for about half of the rows, where the result is that infinity.  So where a row with a finite sum has
    // a non-finite channel, the channel's values are looked up.  Every row reads the prefix's keys and no channel
    // comes out finite with such a value, so testing row tile 0 (products of pairs) tells whether there is anything to look at:
    // testing both took a short call 0.15-0.3 us more (20 rows over 600 keys 10.8 against 10.65, 2 KV heads paged 10.7 against 10.4).
    l_run[0] = sum_over_rows(l_run[0]);
    l_run[1] = sum_over_rows(l_run[1]);
    auto finite = [&](int t) INLINE {
        float x[2] = {0.f, 0.f};
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            x[0] = __builtin_fmaf(acc[t][e][0], acc[t][e][1], x[0]);
            x[1] = __builtin_fmaf(acc[t][e][2], acc[t][e][3], x[1]);
        }
        return __builtin_fabsf(x[0] + x[1]) < INFINITY;
    };
    auto wrong = [&](int t) INLINE { return l_run[t] < INFINITY && !finite(t); };
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!finite(0)) != 0, 0) && __builtin_amdgcn_ballot_w64(wrong(0) || wrong(1)) != 0) {
        // lane l looks at channels CL l .. of the range's prefix keys; bits 3 i of `seen` channel CL l + i: +inf, -inf, NaN
        constexpr int CL = HD / 64;
        uint32_t seen = 0;
        auto look = [&](int k_a, int k_z) INLINE {
            for (int k = k_a; k < k_z; ++k) {
                const char *row = pv + ((size_t)g * Lp + k) * ROWB;
                if constexpr (PAGED) {
                    const int32_t page = scalar_load(a.page_table + uni(min(k / kPageSize, a.max_pages - 1)));
                    if (page < 0 || page >= a.n_pool_pages) continue;
                    row = pv + (((size_t)page * Hkv + g) * kPageSize + k % kPageSize) * ROWB;
                }
#pragma unroll
                for (int i = 0; i < CL; ++i) {
                    const uint32_t x = reinterpret_cast<const uint16_t *>(row)[CL * lane_c + i];
                    seen |= (x == 0x7f80u ? 1u : x == 0xff80u ? 2u : (x & 0x7fffu) > 0x7f80u ? 4u : 0u) << (3 * i);
                }
            }
        };
        look(s0 * KT, (s0 + nmain) * KT);
        if (tail_t0 == 0 && ntot > nmain) look(tail0, Lp);  // (fewer than 64 keys: the first tail tile)
#pragma unroll
        for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = 16 * e + 4 * q4c + j;
                const uint32_t f = (uint32_t)__shfl((int)seen, c / CL) >> (3 * (c % CL)) & 7u;
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    if (l_run[t] < INFINITY && (f == 1 || f == 2)) acc[t][e][j] = f == 1 ? INFINITY : -INFINITY;
            }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const float l = l_run[t];
        const int lr = u * 32 + 16 * t + l16c;
        if (lr >= rows_head) continue;
        const int s = lr / a.split.group, h = g * G + lr - s * G;
        const size_t orow = (size_t)r * rows_total + (size_t)s * Hq + h;
        // a row with no keys in this range: lse = -inf (the merge takes nothing of its o)
        const bool empty = !(l > 0.f) && !(l != l);
        if (q4c == 0) a.part_lse[orow] = empty ? -INFINITY : (__log2f(l) - nm[t]) * kLn2;
        if (empty) continue;
        const float inv = 1.f / l;
        float *dst = a.part_o + orow * HD + 4 * q4c;
#pragma unroll
        for (int e = 0; e < NE; ++e) *reinterpret_cast<f32x4 *>(dst + 16 * e) = acc[t][e] * inv;
    }
}

template <bool PAGED>  // head_dim 128
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void prefill_tiles_kernel(PrefillArgs a)
{
    prefill_tiles<128, PAGED>(a);
}

template <bool PAGED>  // head_dim 64
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void prefill_tiles_d64_kernel(PrefillArgs a)
{
    prefill_tiles<64, PAGED>(a);
}

}  // namespace

int prefill_tiles_unit_rows() { return 32; }
int prefill_tiles_waves() { return NW; }

int prefill_tiles_blocks_per_cu(int head_dim, bool paged)
{
    const void *f = nullptr;
    if (head_dim == 128)
        f = paged ? reinterpret_cast<const void *>(&prefill_tiles_kernel<true>)
                  : reinterpret_cast<const void *>(&prefill_tiles_kernel<false>);
    else if (head_dim == 64)
        f = paged ? reinterpret_cast<const void *>(&prefill_tiles_d64_kernel<true>)
                  : reinterpret_cast<const void *>(&prefill_tiles_d64_kernel<false>);
    int n = 0;
    if (!f || hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, 64 * NW, 0) != hipSuccess) return 0;
    return n;
}

hipError_t launch_prefill_tiles(const PrefillArgs &a, int n_blocks, int head_dim, hipStream_t s)
{
    if (n_blocks <= 0) return hipSuccess;
    if (head_dim == 128) {
        if (a.paged)
            prefill_tiles_kernel<true><<<n_blocks, 64 * NW, 0, s>>>(a);
        else
            prefill_tiles_kernel<false><<<n_blocks, 64 * NW, 0, s>>>(a);
    } else if (head_dim == 64) {
        if (a.paged)
            prefill_tiles_d64_kernel<true><<<n_blocks, 64 * NW, 0, s>>>(a);
        else
            prefill_tiles_d64_kernel<false><<<n_blocks, 64 * NW, 0, s>>>(a);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace fka
