// k_prompt.hip -- prompt-phase significance (Sec. 4) on the matrix cores.
//
// Token p of an N-token prompt is scored by the mean, over the queries
// j = p..N-1, of the causal softmax probability query j gives it, the KV
// head's g query heads combined by their maximum per query.  Two passes over
// the prompt's fp16 q and k, both built on v_mfma_f32_32x32x16_f16 tiles
// (fp16 products, exact in fp32, fp32 sums):
//
//   ps_rows  per (sequence, KV head, 64 query positions): the log2-sum-exp of
//            every query row of the group's heads over keys 0..j.  A wave holds
//            64 queries of one head in registers as MFMA B operands; blocks of
//            64 keys pass through LDS as A operands, so a tile's sixteen logits
//            per lane belong to one query and their sum needs no exchange.  The
//            running max is raised only when a tile's sum passes 2^6 (a
//            wave-uniform branch; a far larger bound would not overflow, but the
//            largest exponents are rounded at their own size: the scores' error
//            against 64 bits is 4.5e-7 with 2^6, 4.8e-7 with 2^8 on 16 prompts of
//            1k-4k tokens), so a logit costs one fma, one exp2, one add.
//   ps_cols  per (sequence, KV head, 256 keys): 64 keys per wave in registers
//            as B operands; tiles of 32 query positions x up to four heads pass
//            through LDS as A operands.  Each tile's accumulation starts at its
//            rows' -lse / c (read from LDS into the accumulator), so the
//            maximum over the heads needs nothing per head and one exp2 gives
//            the group's probability; a lane's sixteen values belong to one
//            key, whose sum stays in the lane to the end: no atomics, a fixed
//            order.  Few key blocks are cut into query segments (prompt_segs).
//
// Both ask for the next tile before they compute one, by loads with an LDS
// destination.  They overlap across waves more than within one: in most instances
// the compiler's first use of the fragments loaded before the loop comes after those
// loads and waits for them too (for any load still counted, as it cannot see the
// wait in the inline asm of stage_ready).  The MFMA results stay in VGPRs (two or three waves per SIMD
// bound the registers to 256; with more, every result went through an AGPR
// copy).
//
// Bound by the matrix cores and, in the row pass, VALU issue about equally (one
// exp2 is two slots): 64 prompts of 1k-4k tokens at 32 / 8 heads, 2 x 1.73
// TFLOP, take 1.95 + 1.98 ms, 880 TFLOP/s, where a large library fp16 product
// reaches 1260 on the device.  With 16x16 tiles through AGPRs, register-staged
// and one workgroup per block it was 2.7 + 2.8 ms; of that, the 32x32 tiles
// gave 0.4 and 0.1, work lists instead of workgroups per block (below) 0.3
// and 0.6.

#include "internal.hpp"

namespace dkv {

namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));

constexpr int kPsThreads = 256;         // 4 waves (offsets and column pass)
constexpr int kKeyBlock = 64;           // keys per LDS stage of the row pass
constexpr int kColKeys = 256;           // keys per workgroup of the column pass (64 per wave)
constexpr int kChunks = 16;             // 16-byte chunks of a 128-half row
constexpr float kRaise = 0x1p6f;        // row pass: a tile's sum past this raises the running max
constexpr float kLog2e = 1.4426950408889634f;

// Row pass: a wave takes 64 query positions of one head, a workgroup all heads
// of kPos positions, or half of seven or eight heads (four waves for one or two
// heads, one wave per head above).  168 VGPRs: three waves per SIMD.
template <int G>
struct RowShape {
    static constexpr int kGroups = G >= 7 ? 2 : 1;               // head groups
    static constexpr int kWaves = G <= 2 || G >= 7 ? 4 : G;
    static constexpr int kPos = G <= 2 ? 64 * (4 / G) : 64;
    static constexpr int kPerCu = 12 / kWaves;                   // resident workgroups per CU
};

// Column pass: a stage in LDS is kTiles tiles of 32 query positions x up to four
// heads (groups of a tile's heads follow each other).
template <int G>
struct ColShape {
    static constexpr int kGroups = (G + 3) / 4;
    static constexpr int kHeads = (G + kGroups - 1) / kGroups;  // heads of a full group
    static constexpr int kTiles = G == 1 ? 4 : (G == 2 ? 2 : 1);
    static constexpr int kUnits = kTiles * kHeads;              // 32-row units of a stage
};

// With a zero addend the compiler may place the result over an operand that is not used
// again.  An earlier kernel whose MFMA results lay over their B operand gave wrong
// scores, so no kernel here relies on what the hardware does then: an operand of such a
// product is named once more after it.
__device__ __forceinline__ f16v mfma32(h8 a, h8 b, f16v c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max(a, b) as the median of a, b and infinity.  The compiler makes it a maximum again and
// at GQ 2, 4, 6, 7 and 8 quiets both operands first (64 to 128 extra instructions in the
// column pass's loop); NaN operands are ignored either way.
__device__ __forceinline__ float max_med(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, __builtin_huge_valf()); }

// Work items: (pair = sequence and KV head, block), in eight lists, one per XCD
// (consecutive workgroups go round-robin over the XCDs, so workgroup i takes item i / 8
// of list i % 8).  List x holds pairs x, x + 8, ..., eight of them at a time (a group),
// block-major with the heaviest block (0) first: the blocks of a pair run close
// together and share its rows in one XCD's L2, and every list has pairs from all
// over the batch.  Which workgroup takes an item does not change its result.
//
// A pass of few items (PromptArgs::once) has a workgroup per item.  The items vary by a
// factor of N in work, and workgroups are dispatched strictly in order, over the
// shader engines in turn: with long prompts one workgroup per item kept 62 % of the
// waves resident (column pass, 64 prompts of 1k-4k tokens).  So in a pass of many items
// each resident workgroup goes on with further items of its list, handed out by a
// counter, then of the others, until there are none; a group there has the blocks of
// its own longest prompt (ps_offsets): with those of the batch's longest for every
// pair most items of one prompt of 4096 and 1023 of 16 tokens were empty (32 / 8 heads:
// 7.6 ms; 2.1 with a workgroup per item, 0.5 so).
struct WorkItems {
    const int* start;  // [kPromptQueues][groups + 1] first item of each group, the list's items last
    int* ctr;          // items handed out beyond the workgroups' first ones
    int once, pairs, groups;
    int nblk;          // blocks of every pair, once
    __device__ __forceinline__ int first_items(int x) const { return ((int)gridDim.x - x + kPromptQueues - 1) / kPromptQueues; }
    __device__ __forceinline__ int items(int x) const { return start[x * (groups + 1) + groups]; }
    // Item k of list x: pair, block, blocks of the pair's group; false past the list's end.  Whole waves.
    __device__ __forceinline__ bool locate(int x, int k, int& pair, int& blk, int& blocks) const
    {
        if (once) {  // all pairs are one group
            const int i = k * kPromptQueues + x;
            blocks = nblk;
            blk = i / pairs;
            pair = i - blk * pairs;
            return true;
        }
        const int* sx = start + x * (groups + 1);
        if (k >= sx[groups]) return false;
        const int lane = threadIdx.x & (kWave - 1);
        int g = 0;
        for (int len = groups; len > 1;) {  // the last group that starts at or before k
            const int step = (len + kWave - 1) / kWave, at = lane * step;
            const int c = __popcll(__builtin_amdgcn_ballot_w64(at < len && sx[g + (at < len ? at : 0)] <= k)) - 1;
            g += c * step;
            len = min(step, len - c * step);
        }
        const int first = sx[g], np = (pairs - x + kPromptQueues - 1) / kPromptQueues;
        const int w = min(kPromptGroup, np - g * kPromptGroup);
        blocks = (sx[g + 1] - first) / w;
        blk = (k - first) / w;
        pair = x + kPromptQueues * (g * kPromptGroup + (k - first) % w);
        return true;
    }
    // The next item to take, from list x on (one whole wave); false: none is left.
    __device__ __forceinline__ bool next(int& x, int& k) const
    {
        const int lane = threadIdx.x & (kWave - 1);
        for (;;) {
            int got = 0;
            if (lane == 0) got = atomicAdd(ctr + x * kPromptCtrStride, 1);
            k = first_items(x) + __builtin_amdgcn_readfirstlane(got);
            if (k < items(x)) return true;
            // which lists have items: all eight counters at once
            bool left = false;
            if (lane < kPromptQueues)
                left = first_items(lane) + __hip_atomic_load(ctr + lane * kPromptCtrStride, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT) < items(lane);
            const unsigned m = (unsigned)__builtin_amdgcn_ballot_w64(left);
            if (!m) return false;
            x = (x + __builtin_ctz(m >> x | m << (kPromptQueues - x))) % kPromptQueues;
        }
    }
};

// f(pair, block, blocks of the pair's group) for the workgroup's items.
template <typename F>
__device__ __forceinline__ void for_items(const WorkItems& wi, F&& f)
{
    __shared__ int s_next[2];
    int x = blockIdx.x % kPromptQueues, k = blockIdx.x / kPromptQueues;
    for (;;) {
        int pair, blk, blocks;
        if (wi.locate(x, k, pair, blk, blocks)) f(pair, blk, blocks);
        if (wi.once) return;
        __syncthreads();  // s_next and the item's LDS are written again
        if (wave_index() == 0) {
            if (!wi.next(x, k)) x = -1;
            if (threadIdx.x == 0) {
                s_next[0] = x;
                s_next[1] = k;
            }
        }
        __syncthreads();
        x = __builtin_amdgcn_readfirstlane(s_next[0]);
        k = __builtin_amdgcn_readfirstlane(s_next[1]);
        if (x < 0) return;
    }
}

// LDS rows of 16 chunks without padding (loads with an LDS destination write
// consecutive lanes' chunks side by side): chunk c of row r sits at c ^ (r % 16),
// so sixteen rows' reads of one chunk fall into different banks.
__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ (row & (kChunks - 1)); }

// Loads with an LDS destination: four rows of 256 bytes, lane l taking the chunk
// that belongs at place l % 16 of row l / 16; the 1 KiB lands at lds.
// By address per lane, or (load_rows_at) uniform address plus a lane's 32-bit
// byte offset.
__device__ __forceinline__ uint32_t lds_addr(const void* lds)
{
    return (uint32_t)(size_t)(__attribute__((address_space(3))) const void*)lds;
}
__device__ __forceinline__ void load_rows(const uint16_t* src, const void* lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr(lds)), "v"(src) : "memory");
}
__device__ __forceinline__ void load_rows_at(const uint16_t* src, uint32_t off, const void* lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr(lds)), "v"(off), "s"(src) : "memory");
}
// Rows 4 * part .. of a tile whose row r starts at base + r * stride (elements;
// rows past `most` repeat it).  v0: the lane's byte offset for part 0, i.e. its
// row l / 16 and place l % 16 (lane_offset); the swizzle of part p is an
// exclusive or with its rows' upper two bits.
__device__ __forceinline__ uint32_t lane_offset(long long stride)
{
    const int lane = threadIdx.x & (kWave - 1);
    return (uint32_t)(lane >> 4) * (uint32_t)(stride * 2) + (uint32_t)((lane & 15) ^ (lane >> 4)) * 16;
}
constexpr long long kMaxStride = 1LL << 28;  // elements per row up to which lane_offset fits 32 bits
__device__ __forceinline__ void load_part(const uint16_t* base, long long stride, int part, int most, uint32_t v0,
                                          const void* lds)
{
    if (most >= 4 * part + 3 && stride <= kMaxStride) {
        load_rows_at(base + 4 * part * stride, v0 ^ (uint32_t)((part & 3) << 6), lds);
    } else {
        const int lane = threadIdx.x & (kWave - 1);
        int r = 4 * part + (lane >> 4);
        asm volatile("" : "+v"(r));  // (computed here: the rare side's addresses stay out of the loops' registers)
        load_rows(base + (long long)min(r, most) * stride + swz(r, lane & 15) * 8, lds);
    }
}
// The loads above are seen by the workgroup: each wave waits for its own, then all meet.
__device__ __forceinline__ void stage_ready()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

}  // namespace

// Row starts and lengths: off[b] = sum of the clamped lengths before b; a
// sequence's rows are cut at total_new, so no pass touches a row >= total_new.
__global__ __launch_bounds__(kPsThreads) void ps_offsets(PromptArgs a)
{
    __shared__ long long part[kPsThreads];
    const int tid = threadIdx.x;
    if (tid < 2 * kPromptQueues) a.ctr[tid * kPromptCtrStride] = 0;
    const int per = (a.B + kPsThreads - 1) / kPsThreads;
    const int b0 = tid * per, b1 = min(a.B, b0 + per);
    long long s = 0;
    for (int b = b0; b < b1; b++) s += min(max(a.new_len[b], 0), a.max_new);
    part[tid] = s;
    __syncthreads();
    for (int d = 1; d < kPsThreads; d <<= 1) {
        const long long v = tid >= d ? part[tid - d] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    long long off = part[tid] - s;
    for (int b = b0; b < b1; b++) {
        const int n = min(max(a.new_len[b], 0), a.max_new);
        const long long room = a.total_new - off;
        a.off[b] = off;
        a.nlen[b] = (int)(room <= 0 ? 0 : (n < room ? n : room));
        off += n;
    }
    if (a.once[0] && a.once[1]) return;
    // first items of every list's groups, for both passes: a wave per list
    __syncthreads();
    const int lane = tid & (kWave - 1), pairs = a.B * a.Hkv;
    for (int x = wave_index(); x < kPromptQueues; x += kPsThreads / kWave) {
        int before[2] = {0, 0};
        for (int g0 = 0; g0 <= a.groups; g0 += kWave) {
            const int g = g0 + lane, p0 = x + kPromptQueues * kPromptGroup * g;
            int n = 0, w = 0;
            if (g < a.groups) {
                for (int j = 0; j < kPromptGroup; j++) {
                    const int p = p0 + kPromptQueues * j;
                    if (p < pairs) {
                        n = max(n, a.nlen[p / a.Hkv]);
                        w++;
                    }
                }
            }
            const int items[2] = {(n + a.row_pos - 1) / a.row_pos * a.row_groups * w,
                                  (n + kColKeys - 1) / kColKeys * a.segs * w};
            for (int i = 0; i < 2; i++) {
                const int incl = wave_incl_scan(items[i]);
                if (g <= a.groups) a.start[(i * kPromptQueues + x) * (a.groups + 1) + g] = before[i] + incl - items[i];
                before[i] += __builtin_amdgcn_readlane(incl, kWave - 1);
            }
        }
    }
}

// Pass 1: lse2[row][hq] = log2 sum_{p <= j} exp2(scale_log2 * q_j . k_p).
// One item: a pair's block of query positions (blk 0 the last, the heaviest).
template <int G>
__device__ __forceinline__ void rows_item(const PromptArgs& a, h8 (&sk)[2][kKeyBlock][kChunks], int bh, int qb, int hg)
{
    using R = RowShape<G>;
    constexpr int kWaves = R::kWaves, PB = R::kPos;
    const int b = bh / a.Hkv, h = bh - b * a.Hkv;
    const int N = __builtin_amdgcn_readfirstlane(a.nlen[b]);
    const long long off = read_lane<long long>(a.off[b], 0);  // (scalar: the loads' base)
    const int q0 = qb * PB;

    const int lane = threadIdx.x & (kWave - 1);
    const int w = wave_index();
    const int col = lane & 31, half = lane >> 5;
    const int t = G == 1 ? 0 : (G == 2 ? (w & 1) : 4 * hg + w);
    const int wq0 = q0 + (G == 1 ? 64 * w : (G == 2 ? 64 * (w >> 1) : 0));
    const float c = a.scale_log2;
    const bool idle = wq0 >= N || t >= G;  // (uniform) this wave only stages keys

    // B operands: 32 positions per block, k = 16 s + 8 half ..
    h8 qf[2][8];
    for (int cb = 0; cb < 2; cb++) {
        // (positions past the prompt repeat its last, heads past the group its last: not written)
        const int j = min(wq0 + 32 * cb + col, N - 1);
        const h8* src = reinterpret_cast<const h8*>(a.q + ((off + j) * a.Hq + h * G + min(t, G - 1)) * kD);
        for (int s = 0; s < 8; s++) qf[cb][s] = src[2 * s + half];
    }
    float m[2] = {-1e30f, -1e30f}, sum[2] = {0.0f, 0.0f};

    const int last = min(N, q0 + PB) - 1;
    const int nkb = last / kKeyBlock + 1;
    const long long stride = (long long)a.Hkv * kD;
    const uint32_t v0 = lane_offset(stride);
    auto stage = [&](int kb) {  // (rows past the prompt repeat its last: masked)
        const uint16_t* base = a.k + ((off + (long long)kb * kKeyBlock) * a.Hkv + h) * kD;
#pragma unroll
        for (int i = 0; i < (16 + kWaves - 1) / kWaves; i++) {
            const int part = i * kWaves + w;
            if (part < 16) load_part(base, stride, part, N - 1 - kb * kKeyBlock, v0, &sk[kb & 1][4 * part][0]);
        }
    };
    stage(0);
    for (int kb = 0; kb < nkb; kb++) {
        stage_ready();
        if (kb + 1 < nkb) stage(kb + 1);
        const int buf = kb & 1;
#pragma unroll
        for (int kt = 0; kt < 2; kt++) {
            const int key0 = kb * kKeyBlock + 32 * kt;
            // (uniform) all of the wave's positions precede the keys
            if (key0 > wq0 + 63 || idle) continue;
            h8 af[8];
            for (int s = 0; s < 8; s++) af[s] = sk[buf][32 * kt + col][swz(col, 2 * s + half)];
            f16v acc[2];
#pragma unroll
            for (int cb = 0; cb < 2; cb++) {
                f16v z;
                for (int i = 0; i < 16; i++) z[i] = 0.0f;
                acc[cb] = mfma32(af[0], qf[cb][0], z);
                asm("" : "+v"(acc[cb]) : "v"(af[0]));  // (see mfma32)
                for (int s = 1; s < 8; s++) acc[cb] = mfma32(af[s], qf[cb][s], acc[cb]);
            }
#pragma unroll
            for (int cb = 0; cb < 2; cb++) {
                const int jb = wq0 + 32 * cb;
                // the diagonal (it also removes keys >= N: they lie after every valid
                // position); the empty asm keeps the selects inside the branch
                if (key0 + 31 > jb) {
                    const int lim = jb + col - key0 - 4 * half;
                    for (int i = 0; i < 16; i++) {
                        float v = 8 * (i / 4) + i % 4 > lim ? -__builtin_huge_valf() : acc[cb][i];
                        asm volatile("" : "+v"(v));
                        acc[cb][i] = v;
                    }
                }
                auto tile_sum = [&]() {
                    const float nm = -m[cb];
                    float s0 = 0.0f, s1 = 0.0f;
                    for (int i = 0; i < 16; i += 2) {
                        s0 += fast_exp2(fmaf(acc[cb][i], c, nm));
                        s1 += fast_exp2(fmaf(acc[cb][i + 1], c, nm));
                    }
                    return s0 + s1;
                };
                float ts = tile_sum();
                if (__builtin_amdgcn_ballot_w64(!(ts <= kRaise))) {
                    float mx = acc[cb][0];
                    for (int i = 1; i < 16; i++) mx = fmaxf(mx, acc[cb][i]);
                    const float mn = fmaxf(m[cb], mx * c);
                    sum[cb] *= fast_exp2(m[cb] - mn);
                    m[cb] = mn;
                    ts = tile_sum();
                }
                sum[cb] += ts;
            }
        }
    }
    // the two halves' keys of each position
    for (int cb = 0; cb < 2; cb++) {
        const int j = wq0 + 32 * cb + col;
        const float mo = __shfl_xor(m[cb], 32), so = __shfl_xor(sum[cb], 32);
        const float mx = fmaxf(m[cb], mo);
        const float sm = sum[cb] * fast_exp2(m[cb] - mx) + so * fast_exp2(mo - mx);
        if (half == 0 && j < N && t < G) a.lse2[(off + j) * a.Hq + h * G + t] = mx + __builtin_amdgcn_logf(sm);
    }
}

template <int G>
__global__ __launch_bounds__(RowShape<G>::kWaves * kWave, 3) void ps_rows(PromptArgs a)
{
    using R = RowShape<G>;
    __shared__ h8 sk[2][kKeyBlock][kChunks];
    const WorkItems wi = {a.start, a.ctr, a.once[0], a.B * a.Hkv, a.groups,
                          (a.max_new + R::kPos - 1) / R::kPos * R::kGroups};
    for_items(wi, [&](int pair, int blk, int blocks) {  // blk 0 the last positions
        const int qb = (blocks - 1 - blk) / R::kGroups;
        if (qb * R::kPos < a.nlen[pair / a.Hkv]) rows_item<G>(a, sk, pair, qb, blk % R::kGroups);
    });
}

// Pass 2: score[row][h] = (1 / (N - p)) sum_{j >= p} max_t exp2(scale_log2 * q_j,t . k_p - lse2[j][t]).
template <int G>
struct ColLds {
    h8 q[2][ColShape<G>::kUnits][32][kChunks];  // [stage][tile * heads + head][position]
    float bias[2][ColShape<G>::kUnits][32];     // -lse / c of those rows
};

// One item: a pair's block of 256 keys (kb 0 the heaviest) and a segment of its
// query tiles.
template <int G>
__device__ __forceinline__ void cols_item(const PromptArgs& a, ColLds<G>& lds, int bh, int kb, int seg)
{
    using S = ColShape<G>;
    constexpr int QI = 32 * S::kTiles;               // query positions per stage
    const int b = bh / a.Hkv, h = bh - b * a.Hkv;
    const int N = __builtin_amdgcn_readfirstlane(a.nlen[b]);
    const long long off = read_lane<long long>(a.off[b], 0);  // (scalar: the loads' base)
    const int k0 = kb * kColKeys;

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int w = wave_index();
    const int col = lane & 31, half = lane >> 5;
    const int wk0 = k0 + w * 64;
    const float c = a.scale_log2;
    const float inv_c = 1.0f / c;

    // B operands: 32 keys per block, k = 16 s + 8 half ..
    h8 kf[2][8];
    for (int cb = 0; cb < 2; cb++) {
        const int p = min(wk0 + 32 * cb + col, N - 1);  // (keys past the prompt repeat its last: not written)
        const h8* src = reinterpret_cast<const h8*>(a.k + ((off + p) * a.Hkv + h) * kD);
        for (int s = 0; s < 8; s++) kf[cb][s] = src[2 * s + half];
    }
    float cs[2] = {0.0f, 0.0f};

    const int nq = (N - k0 + QI - 1) / QI;  // stages [it0, it1) of the segment's positions
    const int it0 = (int)((long long)seg * nq / a.segs), it1 = (int)((long long)(seg + 1) * nq / a.segs);
    float pl = 0.0f;
    bool pl_off = false;
    const float lse_scale = (a.lse ? -kLog2e : -1.0f) * inv_c;
    const long long stride = (long long)a.Hq * kD;
    const uint32_t v0 = lane_offset(stride);
    // Stage s = it * kGroups + g: positions k0 + it * QI .., heads g * kHeads ..
    auto heads_of = [](int g) { return min(S::kHeads, G - g * S::kHeads); };
    auto stage = [&](int it, int g, int buf) {
        const int j0 = k0 + it * QI;
        const int nh = heads_of(g), h0 = g * S::kHeads;
        // (the parts' addresses are formed anew: kept over the loop they spill)
        long long step = stride;
        asm volatile("" : "+s"(step));
        const uint16_t* base = a.q + (off + j0) * step + (h * G + h0) * kD;
#pragma unroll
        for (int i = 0; i < 2 * S::kUnits; i++) {    // eight 1 KiB parts per unit
            const int part = i * 4 + w, u = part >> 3, tile = u / S::kHeads, t = u - tile * S::kHeads;
            if (t >= nh || j0 + 32 * tile >= N) continue;
            // (positions past the prompt repeat its last: their bias is -inf)
            load_part(base + 32 * tile * step + t * kD, step, part & 7, N - 1 - j0 - 32 * tile, v0, &lds.q[buf][u][4 * (part & 7)][0]);
        }
        if (tid < S::kUnits * 32) {
            const int u = tid >> 5, tile = u / S::kHeads, t = u - tile * S::kHeads;
            const int j = j0 + 32 * tile + (tid & 31);
            const long long e = (off + min(j, N - 1)) * a.Hq + h * G + h0 + min(t, nh - 1);
            pl_off = j >= N || t >= nh;
            pl = (a.lse ? a.lse : a.lse2)[e];  // (scaled where it is used: no wait for the loads here)
        }
    };
    // last positions first: the key blocks of one (sequence, KV head), which run at
    // about the same time on one XCD, then read the same queries together
    if (it1 > it0) stage(it1 - 1, 0, 0);
    int buf = 0;
    for (int it = it1 - 1; it >= it0; it--) {
        f16v mx[S::kTiles][2];
#pragma unroll
        for (int g = 0; g < S::kGroups; g++) {
            if (tid < S::kUnits * 32) lds.bias[buf][tid >> 5][tid & 31] = pl_off ? -__builtin_huge_valf() : pl * lse_scale;
            stage_ready();
            if (g + 1 < S::kGroups) stage(it, g + 1, buf ^ 1);
            else if (it > it0) stage(it - 1, 0, buf ^ 1);
#pragma unroll
            for (int tile = 0; tile < S::kTiles; tile++) {
                const int j0 = k0 + it * QI + 32 * tile;
                if (j0 + 31 < wk0 || wk0 >= N || j0 >= N) continue;  // (uniform) no query of the tile reaches the wave's keys
                // A operands: the tile's positions of one head; the accumulation starts at
                // -lse/c, so the maximum over the heads needs no arithmetic per head
#pragma unroll
                for (int t = 0; t < S::kHeads; t++) {
                    if (t >= heads_of(g)) break;
                    const int u = tile * S::kHeads + t;
                    h8 af[8];
                    for (int s = 0; s < 8; s++) af[s] = lds.q[buf][u][col][swz(col, 2 * s + half)];
                    f16v bias;
                    for (int r = 0; r < 4; r++) {
                        const f4 v = *reinterpret_cast<const f4*>(&lds.bias[buf][u][8 * r + 4 * half]);
                        for (int i = 0; i < 4; i++) bias[4 * r + i] = v[i];
                    }
#pragma unroll
                    for (int cb = 0; cb < 2; cb++) {
                        f16v acc = mfma32(af[0], kf[cb][0], bias);
                        for (int s = 1; s < 8; s++) acc = mfma32(af[s], kf[cb][s], acc);
                        if (g == 0 && t == 0) mx[tile][cb] = acc;
                        else
                            for (int i = 0; i < 16; i++) mx[tile][cb][i] = max_med(mx[tile][cb][i], acc[i]);
                    }
                }
                if (g + 1 < S::kGroups) continue;
#pragma unroll
                for (int cb = 0; cb < 2; cb++) {
                    const int p0 = wk0 + 32 * cb;
                    if (j0 < p0 + 31) {  // the diagonal: queries before the key
                        const int lim = p0 + col - j0 - 4 * half;
                        for (int i = 0; i < 16; i++) {
                            float v = 8 * (i / 4) + i % 4 < lim ? -__builtin_huge_valf() : mx[tile][cb][i];
                            asm volatile("" : "+v"(v));
                            mx[tile][cb][i] = v;
                        }
                    }
                    float s0 = 0.0f, s1 = 0.0f;
                    for (int i = 0; i < 16; i += 2) {
                        s0 += fast_exp2(mx[tile][cb][i] * c);
                        s1 += fast_exp2(mx[tile][cb][i + 1] * c);
                    }
                    cs[cb] += s0 + s1;
                }
            }
            buf ^= 1;
        }
    }
    for (int cb = 0; cb < 2; cb++) {
        const float v = cs[cb] + __shfl_xor(cs[cb], 32);
        const int p = wk0 + 32 * cb + col;
        if (half == 0 && p < N) {
            if (a.segs == 1) a.score[(off + p) * a.Hkv + h] = v / (float)(N - p);
            else a.part[((long long)seg * a.total_new + off + p) * a.Hkv + h] = v;
        }
    }
}

template <int G>
__global__ __launch_bounds__(kPsThreads, 2) void ps_cols(PromptArgs a)
{
    __shared__ ColLds<G> lds;
    const WorkItems wi = {a.start + kPromptQueues * (a.groups + 1), a.ctr + kPromptQueues * kPromptCtrStride, a.once[1],
                          a.B * a.Hkv, a.groups, (a.max_new + kColKeys - 1) / kColKeys * a.segs};
    for_items(wi, [&](int pair, int blk, int) {
        if (blk / a.segs * kColKeys < a.nlen[pair / a.Hkv]) cols_item<G>(a, lds, pair, blk / a.segs, blk % a.segs);
    });
}

// The segments' sums of each (row, KV head), in order, over the row's queries.
__global__ __launch_bounds__(kPsThreads) void ps_finish(PromptArgs a)
{
    const int b = blockIdx.y;
    const int N = a.nlen[b];
    const long long n = (long long)N * a.Hkv, base = a.off[b] * a.Hkv, step = a.total_new * a.Hkv;
    for (long long i = (long long)blockIdx.x * kPsThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kPsThreads) {
        float v = 0.0f;
        for (int s = 0; s < a.segs; s++) v += a.part[s * step + base + i];
        a.score[base + i] = v / (float)(N - (int)(i / a.Hkv));
    }
}

namespace {

// Workgroups of a pass: one per item up to `most` times as many as are resident at once
// (per_cu per CU), or while no prompt is long (their items are alike), else as many as
// are resident.  Handing items out costs a round trip to the counters and two barriers per
// item, one workgroup per item the waves that the order of dispatch leaves out.  Row pass,
// at 32 / 8 heads: 64 prompts of 700 tokens, 7 times the resident, 314 us one per item and 338
// handed out; 64 of 1k-4k, 43 times, 5.07 and 4.75 ms.  Column pass: 64 of 700 at 64 / 8
// heads, 6 times, 318 and 302 us; 64 of 1k-4k, 16 times, 4.75 and 4.41 ms; 2000 of 64
// tokens, 31 times, 640 and 686 us with the row pass.
unsigned pass_grid(long long items, int max_new, int most, int cus, int per_cu, int* once)
{
    const long long resident = (long long)cus * per_cu;
    *once = items <= most * resident || (max_new <= 512 && items <= 1 << 22);  // (a launch's threads fit 32 bits)
    return (unsigned)(*once ? items : resident);
}

template <int G>
hipError_t launch_prompt_g(PromptArgs& a, int cus, hipStream_t st)
{
    using R = RowShape<G>;
    const int pairs = a.B * a.Hkv;
    const long long rblk = (a.max_new + R::kPos - 1) / R::kPos, cblk = (a.max_new + kColKeys - 1) / kColKeys;
    if (a.lse == nullptr && pairs * rblk > 0x7fffffffLL) return hipErrorInvalidValue;
    if (pairs * cblk > 0x7fffffffLL) return hipErrorInvalidValue;
    a.row_pos = R::kPos;
    a.row_groups = R::kGroups;
    a.groups = (pairs + kPromptQueues * kPromptGroup - 1) / (kPromptQueues * kPromptGroup);
    const unsigned rgrid = pass_grid(pairs * rblk * R::kGroups, a.max_new, 16, cus, R::kPerCu, &a.once[0]);
    const unsigned cgrid = pass_grid(pairs * cblk * a.segs, a.max_new, 4, cus, 2, &a.once[1]);
    if (a.lse) a.once[0] = 1;  // (no row pass)
    hipError_t e = launch1(ps_offsets, 1, kPsThreads, st, a);
    if (e == hipSuccess && !a.lse) e = launch1(ps_rows<G>, rgrid, R::kWaves * kWave, st, a);
    if (e == hipSuccess) e = launch1(ps_cols<G>, cgrid, kPsThreads, st, a);
    if (e != hipSuccess || a.segs == 1) return e;
    const long long rows = (long long)a.max_new * a.Hkv;
    const unsigned gx = (unsigned)min((rows + kPsThreads - 1) / kPsThreads, 64LL);
    void* args[] = {&a};
    return hipLaunchKernel(reinterpret_cast<const void*>(ps_finish), dim3(gx, (unsigned)a.B), dim3(kPsThreads), args, 0, st);
}

}  // namespace

hipError_t launch_prompt_significance(const PromptArgs& args, int g, hipStream_t st)
{
    PromptArgs a = args;
    if (a.B <= 0 || a.max_new <= 0) return hipSuccess;
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    if (cus < 1) cus = 1;
    switch (g) {
    case 1: return launch_prompt_g<1>(a, cus, st);
    case 2: return launch_prompt_g<2>(a, cus, st);
    case 3: return launch_prompt_g<3>(a, cus, st);
    case 4: return launch_prompt_g<4>(a, cus, st);
    case 5: return launch_prompt_g<5>(a, cus, st);
    case 6: return launch_prompt_g<6>(a, cus, st);
    case 7: return launch_prompt_g<7>(a, cus, st);
    case 8: return launch_prompt_g<8>(a, cus, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace dkv
