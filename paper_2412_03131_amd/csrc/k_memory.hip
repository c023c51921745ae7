// k_memory.hip -- KV compressor, page allocation and free-list compaction
// kernels for gfx950 (DiffKV Sec. 4, Sec. 5.2, Sec. 5.3).
//
// The compressor runs as two launches on the caller's stream:
//   append_classify  one or more workgroups per table: class its new tokens
//                    (quota form by a two-target radix select on the score
//                    bits, or the Algorithm 1 threshold comparisons) and rank
//                    the kept tokens of each section in position order;
//   append_commit    every workgroup derives the plan from the classify
//                    results (page demand per table, one prefix sum over
//                    tables, all-or-nothing check against the free region and
//                    the table width); workgroup 0 writes the new state, and
//                    every wave takes (table, section, page) jobs: resolve the
//                    page ID (new pages from the table's ring region), quantize
//                    each token's 32-dim groups, write the page.
//   append_one       a call of at most one new token per sequence (a decode
//                    step) in one launch: classes, plan and page jobs, the
//                    state written by the last workgroup to finish.
// Allocation alone (alloc_plan + alloc_write) and compaction (compact_count,
// compact_apply) follow the same planning/coordination split:
// per-table work is fully parallel, one prefix sum gives every table a
// disjoint ring region.
#include <type_traits>

#include "internal.hpp"
#include "quant.hpp"

namespace dkv {

// ---------------------------------------------------------------------------
// shared small pieces
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t score_key(float s)
{
    uint32_t u = __float_as_uint(s);
    if (u == 0x80000000u) u = 0;  // -0 == +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ int ceil_div(int a, int b) { return (a + b - 1) / b; }

// ---------------------------------------------------------------------------
// append_classify: table t = b * Hkv + h, block 512.  One workgroup per table, or
// (few tables with long prompts) cls_split of them, each classing a run of its
// table's tiles of 4096 tokens: every one selects the cuts and counts the classes
// of the tiles before its own again, which costs it a read of the scores, where
// one workgroup after the other would rank them (two prompts of 32k tokens, 16
// tables: 53 us in one workgroup per table).
// Thread tid takes tokens tid, tid + 512, ... of a tile, so a wave's scores come
// from neighbouring rows and its ranks from ballots.
// ---------------------------------------------------------------------------
constexpr int kClsThreads = 512;
static_assert(kClsThreads >= 2 * kWave, "two waves scan the digit histograms");
constexpr int kClsPer = 8;                       // tokens per thread in one tile
static_assert(4 * kClsPer <= 32, "a thread keeps four flag bits per token of a tile in one 32-bit word");
constexpr int kClsTile = kClsThreads * kClsPer;  // the first tile's scores stay in registers
constexpr int kClsWaves = kClsThreads / kWave;
static_assert(kClsPer * kClsWaves == kWave, "a wave scans a tile's counts");
constexpr int kClsBusyGroups = 512;  // workgroups that keep the device busy (two per CU of 256)
static_assert(kClsTile < 65536, "16-bit counts");
constexpr uint32_t kOffSat = 1u << 30;           // row offsets saturate here (above any total_new)

// Sum over the wave of values <= kOffSat, saturating at kOffSat (result in lane 63).
__device__ __forceinline__ uint32_t wave_sat_sum(uint32_t x)
{
    x = min(x + dpp_u32<0x111, 0xF>(x), kOffSat);
    x = min(x + dpp_u32<0x112, 0xF>(x), kOffSat);
    x = min(x + dpp_u32<0x114, 0xF>(x), kOffSat);
    x = min(x + dpp_u32<0x118, 0xF>(x), kOffSat);
    x = min(x + dpp_u32<0x142, 0xA>(x), kOffSat);
    x = min(x + dpp_u32<0x143, 0xC>(x), kOffSat);
    return (uint32_t)__builtin_amdgcn_readlane((int)x, kWave - 1);
}

// Class of one new token against the two cuts of Sec. 4.2 (the high set, and
// the high + low set).  Per cut: a = above it outright, e = tied with the cut
// key (only the first `need` ties in position order are above it).
// mode 0: nothing above the cut, 1: every non-window token, 2: cut at key K.
struct Cuts {
    int mode[2];
    uint32_t K[2];
    int need[2];
};

// PER: tokens per thread in one tile: kClsPer, or one where no sequence has more tokens than
// the workgroup threads (8 tokens to 128 tables: 14.6 -> 14.0 us for the call).
template <int PER>
__global__ __launch_bounds__(kClsThreads) void append_classify(AppendArgs a)
{
    constexpr int kTile = kClsThreads * PER;
    const int H = a.Hkv, NT = a.B * H;
    const int split = blockIdx.x / NT, t = blockIdx.x - split * NT;
    const int b = t / H, h = t - b * H;
    const int tid = threadIdx.x;
    __shared__ long long s_cnt[2][PER * kClsWaves];  // a tile's class counts by step and wave, in position order
    __shared__ int s_before[4];                          // class counts of the tiles before this workgroup's
    __shared__ int s_hist[2][2][256];  // [buffer][cut][digit]
    __shared__ int s_sel[4];
    __shared__ uint32_t s_off;

    if (t == 0 && split == 0 && tid == 0) {  // ring pointers before this call (the commit kernel moves head)
        a.flags->head_old = a.ring_ptr[0];
        a.flags->tail_old = a.ring_ptr[1];
    }
    for (int i = tid; i < 512; i += kClsThreads) (&s_hist[0][0][0])[i] = 0;
    if (tid < 4) s_before[tid] = 0;
    // row offset of this sequence: sum of new_len over lower sequences (wave 0).
    // Entries are clamped to [0, kOffSat] and the sum saturates: a call with an
    // entry outside [0, max_new] fails anyway (that table flags itself).
    if (tid < kWave) {
        uint32_t part = 0;
        for (int i = tid; i < b; i += kWave) {
            const int v = a.new_len[i];
            part = min(part + (uint32_t)(v < 0 ? 0 : (v > (int)kOffSat ? (int)kOffSat : v)), kOffSat);
        }
        part = wave_sat_sum(part);
        if (tid == 0) s_off = part;
    }
    const int n = a.new_len[b];
    TState* ts = a.tstate + t;
    if (split == 0 && tid == 0) {  // section lengths and pages before this call
        ts->lold[0] = a.len[2 * t];
        ts->lold[1] = a.len[2 * t + 1];
        ts->pold[0] = a.pages[2 * t];
        ts->pold[1] = a.pages[2 * t + 1];
    }
    const bool quota = a.quota != nullptr;
    int q0 = 0, q1 = 0;
    if (quota) {
        q0 = a.quota[2 * t];
        q1 = a.quota[2 * t + 1];
    }
    __syncthreads();
    const long long off_b = s_off;
    const bool bad = n < 0 || n > a.max_new || off_b + n > a.total_new ||
                     (b == a.B - 1 && off_b + n != a.total_new);
    if (bad) {
        if (split == 0 && tid == 0) {  // the commit kernel turns n < 0 into DIFFKV_ST_BAD_INPUT
            ts->cnt[0] = ts->cnt[1] = 0;
            ts->n = -1;
        }
        return;
    }
    // this workgroup's tiles [c0, c1) of the table's
    const int tiles = n > kTile ? (n + kTile - 1) / kTile : 1;
    const int per = (tiles + a.cls_split - 1) / a.cls_split;
    const int c0 = split * per, c1 = c0 + per < tiles ? c0 + per : tiles;
    if (c0 >= tiles) return;
    if (h == 0 && split == 0 && tid == 0) {
        a.sold[b] = a.seq_len[b];
        a.row_off[b] = (int)off_b;
    }
    const int W = a.window < n ? a.window : n;
    const int avail = n - W;
    const float* sc = a.score + off_b * H + h;
    int32_t* ord = a.ord + off_b * H + (long long)h * n;

    // scores of step i .. of a tile from `base` on, PER steps' loads together
    auto load_scores = [&](int base, float (&v)[PER]) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int j = base + i * kClsThreads + tid;
            v[i] = j < avail ? sc[(long long)j * H] : 0.f;
        }
    };
    float sr[PER];  // the first tile's stay in registers
    load_scores(0, sr);

    Cuts c = {{0, 0}, {0, 0}, {0, 0}};
    float thr_h = 0.f, thr_l = 0.f;
    if (quota) {
        const int nh = q0 < 0 ? 0 : (q0 > avail ? avail : q0);
        const int nl = q1 < 0 ? 0 : (q1 > avail - nh ? avail - nh : q1);
        const int cut[2] = {nh, nh + nl};
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) c.mode[s2] = cut[s2] <= 0 ? 0 : (cut[s2] >= avail ? 1 : 2);
        if (c.mode[0] == 2 || c.mode[1] == 2) {
            // two-target radix select (the cut[s]-th largest key), 8-bit digits
            // from the top; histograms double-buffered so each digit costs two barriers
            uint32_t prefix[2] = {0, 0}, mask = 0;
            int kk[2] = {c.mode[0] == 2 ? cut[0] : 0, c.mode[1] == 2 ? cut[1] : 0};
            uint32_t kr[PER];
#pragma unroll
            for (int i = 0; i < PER; ++i) kr[i] = score_key(sr[i]);
#pragma unroll
            for (int pass = 0; pass < 4; ++pass) {
                const int shift = 24 - 8 * pass;
                int* hist = &s_hist[pass & 1][0][0];
                auto digits = [&](int base, const uint32_t (&k8)[PER]) {
#pragma unroll
                    for (int i = 0; i < PER; ++i) {
                        if (base + i * kClsThreads + tid < avail) {
                            const uint32_t key = k8[i];
                            const uint32_t dig = (key >> shift) & 255u;
#pragma unroll
                            for (int s2 = 0; s2 < 2; ++s2)
                                if (kk[s2] > 0 && (key & mask) == prefix[s2]) atomicAdd(&hist[s2 * 256 + dig], 1);
                        }
                    }
                };
                digits(0, kr);
                for (int base = kTile; base < avail; base += kTile) {  // beyond the first tile
                    float v[PER];
                    load_scores(base, v);
                    uint32_t k8[PER];
#pragma unroll
                    for (int i = 0; i < PER; ++i) k8[i] = score_key(v[i]);
                    digits(base, k8);
                }
                for (int i = tid; i < 512; i += kClsThreads) (&s_hist[(pass + 1) & 1][0][0])[i] = 0;  // the next digit's buffer
                __syncthreads();
                if (tid < 2 * kWave) {  // two waves find the cut bins with a scan from the top
                    const int s2 = tid / kWave, l = tid & (kWave - 1);
                    if (kk[s2] > 0) {
                        // lane l owns bins 255-4l .. 252-4l (descending)
                        int cb[4], tot4 = 0;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            cb[q] = hist[s2 * 256 + 255 - 4 * l - q];
                            tot4 += cb[q];
                        }
                        const int incl = wave_incl_scan(tot4);
                        int above = incl - tot4;
                        if (above < kk[s2] && incl >= kk[s2]) {
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                if (above + cb[q] >= kk[s2]) {
                                    s_sel[2 * s2] = 255 - 4 * l - q;
                                    s_sel[2 * s2 + 1] = above;
                                    break;
                                }
                                above += cb[q];
                            }
                        }
                    }
                }
                __syncthreads();
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    if (kk[s2] > 0) {
                        prefix[s2] |= (uint32_t)s_sel[2 * s2] << shift;
                        kk[s2] -= s_sel[2 * s2 + 1];
                    }
                }
                mask |= 255u << shift;
            }
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                if (c.mode[s2] == 2) {
                    c.K[s2] = prefix[s2];
                    c.need[s2] = kk[s2];  // tokens with key == K that still belong above the cut
                }
            }
        }
    } else {
        const float N = (float)(a.seq_len[b] + n);
        thr_h = a.alpha_h / N;
        thr_l = a.alpha_l / N;
    }

    // ---- classes and in-section ranks, in position order ------------------
    // Flags of a token: above cut 0, tied at cut 0, above cut 1, tied at cut 1.
    // The high set is the cut-0 set; the low set is the cut-1 set minus it (cut
    // 1's set contains cut 0's), so a token's rank in either follows from the
    // four counts before it.
    auto flags_of = [&](int j, float s) -> uint32_t {
        if (j >= n) return 0u;
        if (j >= avail) return 5u;  // recent window: always high
        if (quota) {
            const uint32_t key = score_key(s);
            const uint32_t f0 = c.mode[0] == 1 ? 1u : (c.mode[0] == 2 ? (uint32_t)(key > c.K[0]) | ((uint32_t)(key == c.K[0]) << 1) : 0u);
            const uint32_t f1 = c.mode[1] == 1 ? 1u : (c.mode[1] == 2 ? (uint32_t)(key > c.K[1]) | ((uint32_t)(key == c.K[1]) << 1) : 0u);
            return f0 | (f1 << 2);
        }
        const uint32_t a0 = s >= thr_h, a1 = a0 | (uint32_t)(s >= thr_l);
        return a0 | (a1 << 2);
    };
    const int wave = wave_index(), lane = lane_id();
    const uint64_t below = (1ull << lane) - 1ull;
    int c_f[4] = {0, 0, 0, 0};  // counts before the tile
    if (c0 > 0) {
        int mine[4] = {0, 0, 0, 0};  // (uniform) this wave's
        for (int base = 0; base < c0 * kTile; base += kTile) {
            float v[PER];
            load_scores(base, v);
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const uint32_t f = flags_of(base + i * kClsThreads + tid, v[i]);
#pragma unroll
                for (int q = 0; q < 4; ++q) mine[q] += __popcll(__builtin_amdgcn_ballot_w64(f >> q & 1u));
            }
        }
        if (lane < 4) atomicAdd(&s_before[lane], lane == 0 ? mine[0] : (lane == 1 ? mine[1] : (lane == 2 ? mine[2] : mine[3])));
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) c_f[q] = s_before[q];
    }
    for (int ct = c0; ct < c1; ++ct) {
        const int base = ct * kTile;
        float v[PER];
        if (ct > 0) {
            load_scores(base, v);
        } else {
#pragma unroll
            for (int i = 0; i < PER; ++i) v[i] = sr[i];
        }
        // per step and wave the four counts, 16 bits each (a tile has 4096 tokens)
        uint32_t fl = 0;  // four flag bits per token
        long long* cnt = s_cnt[ct & 1];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint32_t f = flags_of(base + i * kClsThreads + tid, v[i]);
            fl |= f << (4 * i);
            long long p = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) p |= (long long)__popcll(__builtin_amdgcn_ballot_w64(f >> q & 1u)) << (16 * q);
            if (lane == 0) cnt[i * kClsWaves + wave] = p;
        }
        __syncthreads();  // (the other buffer is free again: every wave has passed its last barrier's reads)
        const long long own = lane < PER * kClsWaves ? cnt[lane] : 0;
        const long long incl = wave_incl_scan64(own), excl = incl - own;  // (no carry between the 16-bit fields)
        const long long tot = read_lane<long long>(incl, kWave - 1);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (base + i * kClsThreads >= n) break;  // (uniform)
            const uint32_t f = fl >> (4 * i);
            const long long ex = read_lane<long long>(excl, i * kClsWaves + wave);
            int r[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                r[q] = c_f[q] + (int)(ex >> (16 * q) & 0xffff) + __popcll(__builtin_amdgcn_ballot_w64(f >> q & 1u) & below);
            const int j = base + i * kClsThreads + tid;
            const int rh = r[0] + min(r[1], c.need[0]);  // high tokens before this one
            const int rt = r[2] + min(r[3], c.need[1]);  // high + low tokens before it
            // (the ranks stay inside the table's n slots; the bounds tests only guard memory)
            if ((f & 1u) || ((f & 2u) && r[1] < c.need[0])) {
                if (rh < n) ord[rh] = j;
            } else if ((f & 4u) || ((f & 8u) && r[3] < c.need[1])) {
                if ((unsigned)(rt - rh) < (unsigned)n) ord[n - 1 - (rt - rh)] = j;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) c_f[q] += (int)(tot >> (16 * q) & 0xffff);
    }
    if (tid == 0 && c1 == tiles) {
        const int hi = c_f[0] + min(c_f[1], c.need[0]);
        ts->cnt[0] = hi;
        ts->cnt[1] = c_f[2] + min(c_f[3], c.need[1]) - hi;
        ts->n = n;
    }
}

constexpr int kPlanThreads = 1024;

// ---------------------------------------------------------------------------
// append_commit: plan + quantize in one launch.
// Every workgroup first derives the call's plan from the per-table state the
// classify kernel left (new tokens per section, section lengths and pages
// before the call): page demand, page jobs, one prefix sum over tables (ring
// region and first job of every table), and the all-or-nothing checks.  So no
// workgroup waits on another: workgroup 0 writes the new state (lengths,
// pages, seq_len, ring head) while all of them -- reading only the snapshot
// -- take page jobs (table, section, page) in job order.
// ---------------------------------------------------------------------------
constexpr int kQuantWaves = kAppendJobsPerGroup;  // page jobs a workgroup runs side by side, one per wave
constexpr int kCommitThreads = kQuantWaves * kWave;
constexpr int kCommitWaves = 4;  // waves per SIMD; whole prefills of 64 prompts of 1k-4k tokens: 3 171, 4 171, 5 (spills) 188 us

// Few jobs go to a whole workgroup each: a wave alone takes a page's slots in up to eight
// steps one after the other, and with a wave or two per SIMD that chain is the call (16
// tokens to each of 128 tables: 14.5 us with four waves per token before the page jobs, 19.6
// with a wave per page, 15.0 so).  The line lies by the bound on the jobs, four per table and the
// tokens' own: up to 1024 (a wave per SIMD), or 2048 of longer appends (33 tokens to 256
// tables, 1816: 16.9 and 20.5 us; but 4 tokens to 384, 1680: 17.9 and 16.9).
constexpr int kCommitFewJobs = 1024;
constexpr int kCommitFewTokens = 8;

struct TablePlan {
    int need[2], jobs[2];
    bool held_over;  // more pages than p_max after the call
};

// Pages hold a power of two of tokens, so page indices are shifts; tsh packs
// the two sections' shifts (high section in bits 0-7, low in bits 8-15).
__device__ __forceinline__ int page_of(int x, int sec, int tsh) { return x >> (sec ? tsh >> 8 : tsh & 255); }

__device__ __forceinline__ TablePlan table_plan(const TState& s, int P, int tsh)
{
    TablePlan tp;
    int held = 0;
#pragma unroll
    for (int sec = 0; sec < 2; ++sec) {
        const int T = 1 << (sec ? tsh >> 8 : tsh & 255);
        const int want = page_of(s.lold[sec] + s.cnt[sec] + T - 1, sec, tsh);
        tp.need[sec] = want > s.pold[sec] ? want - s.pold[sec] : 0;
        held += want > s.pold[sec] ? want : s.pold[sec];
        tp.jobs[sec] =
            s.cnt[sec] ? page_of(s.lold[sec] + s.cnt[sec] - 1, sec, tsh) - page_of(s.lold[sec], sec, tsh) + 1 : 0;
    }
    tp.held_over = held > P;
    return tp;
}

__device__ __forceinline__ long long plan_word(const TablePlan& tp)  // new pages | jobs << 32
{
    return (long long)(tp.need[0] + tp.need[1]) | ((long long)(tp.jobs[0] + tp.jobs[1]) << 32);
}

struct JobDesc {
    int t, sec, p, u0, u1, lold, n, tslot;
    long long ring_idx;  // ring position of a new page, -1 for a page already held
    // one-token append: the sequence's row offset and length before the call
    // come with the job (no classify results); otherwise `one` is 0
    int one, off_b, sold;
};

// Job `job` of table t (its plan tp, its exclusive prefix pre = new pages |
// jobs << 32): section, page, token range, table slot and, for a new page, the
// ring index (the table's ring region, high pages first).
__device__ __forceinline__ void describe_job(JobDesc& d, int t, const TState& s, const TablePlan& tp,
                                             long long pre, int job, int P, long long head_old, int tsh)
{
    const int lj = job - (int)(pre >> 32);
    const int sec = lj < tp.jobs[0] ? 0 : 1;
    const int TT = 1 << (sec ? tsh >> 8 : tsh & 255);
    const int p = page_of(s.lold[sec], sec, tsh) + (sec ? lj - tp.jobs[0] : lj);
    const int lo = s.lold[sec], hi_end = s.lold[sec] + s.cnt[sec];
    d.t = t;
    d.sec = sec;
    d.p = p;
    d.u0 = lo > p * TT ? lo : p * TT;
    d.u1 = hi_end < (p + 1) * TT ? hi_end : (p + 1) * TT;
    d.lold = lo;
    d.n = s.n;
    d.tslot = sec ? P - 1 - p : p;
    d.ring_idx = p < s.pold[sec] ? -1 : head_old + (pre & 0xffffffffll) + (sec ? tp.need[0] : 0) + (p - s.pold[sec]);
    d.one = 0;
    d.off_b = 0;
    d.sold = 0;
}

// The image of one page, as the job composes it in LDS.
constexpr int kPageMax = 4736;  // largest page of the layouts
constexpr bool page_max_covers(int li) { return li >= kNumLayouts || (layout_page_bytes(li) <= kPageMax && page_max_covers(li + 1)); }
static_assert(page_max_covers(0), "page image");
struct PageImage {
    uint4 b[kPageMax / 16];
};

// Eight fp16 values of the caller's k or v, which may start anywhere an fp16 value may:
// still one 16-byte load (the device takes unaligned ones), but never assumed aligned.
typedef uint32_t Fp16x8 __attribute__((ext_vector_type(4), aligned(2)));

// One page job, by JW waves (one, or a whole workgroup, which meets in sync()):
// resolve the page ID (a new page from the table's ring region), quantize the job's tokens, write them, zero a fresh page's
// unused bytes.  Lane = (row of 16, eight dims): row r takes the TT/4 page
// slots from r * TT/4 on, one per step, so a token's key or value vector is one
// 16-byte load per lane, a quad holds a 32-dim group, and a lane ends with its
// dims' codes of TT/4 neighbouring slots, one piece of each dimension-major
// value row (of JW waves each takes its part of the steps, and the pieces are or-ed
// together).  The page is composed in LDS and written in 16-byte pieces: a fresh
// page whole, a continued one by its new slots (its value rows or-ed with the
// old).
// Bound by HBM on bulk appends (fp16 rows in, pages out): 132 us for 64 prompts
// of 1k-4k tokens at 8 KV heads (1.3M token-heads, 60 % kept, 0.55 GB: 4.2 TB/s
// where a large copy reaches 5.1).  One wave per token with two values per
// lane, its codes stored where they fell, took 576 us: about 250 instructions
// per token, most of them for the sixteenfold group extremes and scale.
template <int KB, int VB, int TT, int JW>
__device__ __forceinline__ void commit_job_fmt(const AppendArgs& a, const JobDesc& job, PageImage& img_)
{
    constexpr int kLbK = (1 << KB) - 1, kLbV = (1 << VB) - 1;
    constexpr int NS = TT / 4;                  // slots per row of lanes
    constexpr int NW = NS / JW;                 // and per wave of the job
    constexpr int kStep = JW > 1 ? NW : 2;      // slots per row loaded at once (four: 128 VGPRs and spills)
    constexpr int kAcc = NW * VB > 24 ? 2 : 1;  // value codes of NW slots: exact in one or two floats
    constexpr int kPer = NW / kAcc;
    constexpr int kThr = JW * kWave;
    constexpr int kVBytes = kD * TT * VB / 8;
    const int lane = threadIdx.x & (kWave - 1);
    const int row = lane >> 4, l16 = lane & 15;
    const int jw = JW > 1 ? wave_index() : 0, tid = jw * kWave + lane;  // wave and thread of the job
    auto sync = [] {
        if constexpr (JW > 1) __syncthreads();
        else wave_lds_sync();
    };
    const int P = a.p_max, H = a.Hkv, sec = job.sec;
    const int t = job.t, b = t / H, h = t - b * H;
    uint8_t* img = reinterpret_cast<uint8_t*>(&img_);
    // the page ID, beside the token loads
    int32_t* trow = a.page_table + (long long)t * P;
    int id = job.ring_idx < 0 ? trow[job.tslot] : a.ring[job.ring_idx % a.num_pages];
    const int off_b = job.one ? job.off_b : a.row_off[b];
    const int sold = job.one ? job.sold : a.sold[b];
    // slots [s0, s1) are the job's; lane s < TT: the token of slot s, row
    // ord[u - lold] of its sequence (high, rank order) or ord[n - 1 - (u - lold)]
    // (low ranks are stored from the back); other lanes repeat slot s0's
    const int s0 = job.u0 - job.p * TT, s1 = job.u1 - job.p * TT;
    const bool mine = lane >= s0 && lane < s1;
    int j = 0;
    if (!job.one) {
        const int32_t* ord = a.ord + (long long)off_b * H + (long long)h * job.n;
        const int r = job.p * TT + (mine ? lane : s0) - job.lold;
        j = ord[sec ? job.n - 1 - r : r];
    }
    const float score = a.score[(long long)(off_b + j) * H + h];
    // (uniform) some row's slot of step i is the job's
    auto step_on = [&](int i) { return s1 - s0 >= NS || ((i - s0) & (NS - 1)) < s1 - s0; };
    uint4 kx[kStep], vx[kStep];
    auto load_steps = [&](int i0) {
#pragma unroll
        for (int i = 0; i < kStep; ++i) {
            kx[i] = vx[i] = make_uint4(0, 0, 0, 0);
            if (step_on(i0 + i)) {
                const int jt = __shfl(j, NS * row + i0 + i, kWave);
                const long long at = ((long long)(off_b + jt) * H + h) * (kD / 8) + l16;
                kx[i] = __builtin_bit_cast(uint4, reinterpret_cast<const Fp16x8*>(a.k)[at]);
                vx[i] = __builtin_bit_cast(uint4, reinterpret_cast<const Fp16x8*>(a.v)[at]);
            }
        }
    };
    load_steps(jw * NW);
    id = __builtin_amdgcn_readfirstlane(id);
    if (tid == 0 && job.ring_idx >= 0) trow[job.tslot] = id;
    const int off_kc = a.off_kcode[sec], off_km = a.off_kmeta[sec];
    const int off_vc = a.off_vcode[sec], off_vm = a.off_vmeta[sec];
    const int off_sc = a.off_score[sec], off_pos = a.off_pos[sec];
    const bool fresh = s0 == 0;
    const bool page_ok = (unsigned)id < (unsigned)a.num_pages;  // never write outside the pool
    uint8_t* pg = a.pool + (long long)(page_ok ? id : 0) * a.page_bytes;
    // a page being continued keeps its earlier tokens' value code bits
    constexpr int kVold = (kVBytes + 16 * kThr - 1) / (16 * kThr);
    uint4 vold[kVold];
#pragma unroll
    for (int i = 0; i < kVold; ++i) {
        const int o = 16 * (i * kThr + tid);
        vold[i] = !fresh && o < kVBytes ? *reinterpret_cast<const uint4*>(pg + off_vc + o) : make_uint4(0, 0, 0, 0);
    }
    if (fresh)  // zero what no token covers: of a full page, the bytes past its segments
        for (int o = (s1 < TT ? 0 : off_pos / 16 + TT / 4) + tid; o < (int)a.page_bytes / 16; o += kThr)
            img_.b[o] = make_uint4(0, 0, 0, 0);
    if constexpr (JW > 1)  // the waves' value codes are or-ed together
        if (!fresh || s1 == TT)
            for (int o = tid; o < kVBytes / 16; o += kThr) img_.b[off_vc / 16 + o] = make_uint4(0, 0, 0, 0);
    sync();
    float vrow[kAcc][8];
#pragma unroll
    for (int q = 0; q < kAcc; ++q)
#pragma unroll
        for (int d = 0; d < 8; ++d) vrow[q][d] = 0.0f;
#pragma unroll 1
    for (int i0 = jw * NW; i0 < (jw + 1) * NW; i0 += kStep) {
        if (i0 > jw * NW) load_steps(i0);
#pragma unroll
        for (int i = 0; i < kStep; ++i) {
            if (!step_on(i0 + i)) continue;
            const int sl = NS * row + i0 + i;
            const bool on = sl >= s0 && sl < s1;
            uint32_t ksz, vsz;
            float c[8];
            quant_oct<kLbK>(kx[i], ksz, c);
            if (on) {
                auto f = [](float x, float m, float y) { return __builtin_fmaf(x, m, y); };
                if constexpr (KB == 8) {  // bytes 8 * (l16 & 1) .. of chunk l16 / 2
                    uint2 w;
                    w.x = (uint32_t)f(c[1], 256.0f, c[0]) | (uint32_t)f(c[3], 256.0f, c[2]) << 16;
                    w.y = (uint32_t)f(c[5], 256.0f, c[4]) | (uint32_t)f(c[7], 256.0f, c[6]) << 16;
                    *reinterpret_cast<uint2*>(img + off_kc + ((l16 >> 1) * TT + sl) * 16 + 8 * (l16 & 1)) = w;
                } else {  // bytes 4 * (l16 & 3) .. of chunk l16 / 4
                    const uint32_t w = (uint32_t)f(f(f(c[3], 16.0f, c[2]), 16.0f, c[1]), 16.0f, c[0]) |
                                       (uint32_t)f(f(f(c[7], 16.0f, c[6]), 16.0f, c[5]), 16.0f, c[4]) << 16;
                    *reinterpret_cast<uint32_t*>(img + off_kc + ((l16 >> 2) * TT + sl) * 16 + 4 * (l16 & 3)) = w;
                }
            }
            quant_oct<kLbV>(vx[i], vsz, c);
            const float place = on ? (float)(1 << VB * ((i0 + i) % kPer)) : 0.0f;
#pragma unroll
            for (int q = 0; q < kAcc; ++q) {
                const float at = (i0 + i - jw * NW) / kPer == q ? place : 0.0f;
#pragma unroll
                for (int d = 0; d < 8; ++d) vrow[q][d] = __builtin_fmaf(c[d], at, vrow[q][d]);
            }
            if (on && (l16 & 3) == 0) {
                *reinterpret_cast<uint32_t*>(img + off_km + (sl * kNG + (l16 >> 2)) * 4) = ksz;
                *reinterpret_cast<uint32_t*>(img + off_vm + ((l16 >> 2) * TT + sl) * 4) = vsz;
            }
        }
    }
    // value rows: the piece of slots NS*row + NW*jw .. of dims 8*l16 ..
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        uint8_t* at = img + off_vc + (8 * l16 + d) * (TT * VB / 8);
        if constexpr (JW > 1) {
            const int bit = (row * NS + jw * NW) * VB;
            static_assert(kAcc == 1 && 32 % (NW * VB) == 0, "a wave's codes lie in one word");
            atomicOr(reinterpret_cast<uint32_t*>(at + (bit >> 5) * 4), (uint32_t)vrow[0][d] << (bit & 31));
        } else if constexpr (NS * VB == 32) {
            *reinterpret_cast<uint32_t*>(at + row * 4) = (uint32_t)vrow[0][d] | (uint32_t)vrow[kAcc - 1][d] << 16;
        } else if constexpr (NS * VB == 16) {
            *reinterpret_cast<uint16_t*>(at + row * 2) = (uint16_t)(uint32_t)vrow[0][d];
        } else {
            static_assert(NS * VB == 8, "value row pieces");
            at[row] = (uint8_t)(uint32_t)vrow[0][d];
        }
    }
    if (mine && jw == 0) {
        *reinterpret_cast<float*>(img + off_sc + 4 * lane) = score;
        *reinterpret_cast<int32_t*>(img + off_pos + 4 * lane) = sold + j;
    }
    sync();
    if (page_ok && fresh) {
        for (int o = tid; o < (int)a.page_bytes / 16; o += kThr) reinterpret_cast<uint4*>(pg)[o] = img_.b[o];
    } else if (page_ok) {
        const int ns = s1 - s0;
        for (int i = tid; i < (KB + 1) * ns; i += kThr) {  // key chunks, then key metadata
            const int c = i / ns, sl = s0 + (i - c * ns);
            const int o = c < KB ? off_kc + (c * TT + sl) * 16 : off_km + sl * 16;
            *reinterpret_cast<uint4*>(pg + o) = *reinterpret_cast<const uint4*>(img + o);
        }
        for (int i = tid; i < (kNG + 2) * ns; i += kThr) {  // value metadata, score, position
            const int g = i / ns, sl = s0 + (i - g * ns);
            const int o = g < kNG ? off_vm + (g * TT + sl) * 4 : (g == kNG ? off_sc : off_pos) + sl * 4;
            *reinterpret_cast<uint32_t*>(pg + o) = *reinterpret_cast<const uint32_t*>(img + o);
        }
#pragma unroll
        for (int i = 0; i < kVold; ++i) {
            const int o = off_vc + 16 * (i * kThr + tid);
            if (16 * (i * kThr + tid) >= kVBytes) break;
            const uint4 v = *reinterpret_cast<const uint4*>(img + o);
            *reinterpret_cast<uint4*>(pg + o) = make_uint4(v.x | vold[i].x, v.y | vold[i].y, v.z | vold[i].z, v.w | vold[i].w);
        }
    }
    sync();  // the image is reused by the next job
}

// One page job in the page format of its section (the layouts' formats; see
// kLayoutFmts), so that row widths and bit positions are constants.
template <int JW>
__device__ __forceinline__ void commit_job(const AppendArgs& a, const JobDesc& job, PageImage& img)
{
    const int sec = job.sec;
    const int kb = a.kb[sec], vb = a.vb[sec], T = a.T[sec];
    if (kb == 8 && vb == 4) commit_job_fmt<8, 4, 16, JW>(a, job, img);
    else if (kb == 4 && vb == 2 && T == 32) commit_job_fmt<4, 2, 32, JW>(a, job, img);
    else if (kb == 8 && vb == 8) commit_job_fmt<8, 8, 16, JW>(a, job, img);
    else if (kb == 8 && vb == 2) commit_job_fmt<8, 2, 16, JW>(a, job, img);
    else if (kb == 4 && vb == 1) commit_job_fmt<4, 1, 32, JW>(a, job, img);
    else commit_job_fmt<4, 2, 16, JW>(a, job, img);
}

// A table's state before the call, t uniform: through scalar loads (the
// classify kernel wrote it; no kernel that reads it writes it).
__device__ __forceinline__ TState uniform_state(const TState* ts, int t)
{
    typedef const __attribute__((address_space(4))) int32_t* cptr;
    const cptr p = (cptr)(ts + t);
    TState s;
    s.cnt[0] = p[0];
    s.cnt[1] = p[1];
    s.lold[0] = p[2];
    s.lold[1] = p[3];
    s.pold[0] = p[4];
    s.pold[1] = p[5];
    s.ring_off = p[6];
    s.n = p[7];
    return s;
}

constexpr int kPlanKeep = 2;  // tables per thread whose state stays in registers

// JW: waves of a job, one, or all four of the workgroup where there are few jobs
// (kCommitFewJobs).
template <int JW>
__global__ __launch_bounds__(kCommitThreads, kCommitWaves) void append_commit(AppendArgs a)
{
    const int tid = threadIdx.x;
    const int NT = a.B * a.Hkv;
    const int P = a.p_max;
    __shared__ long long s_scan[kCommitThreads / kWave];
    __shared__ uint32_t s_bits[kCommitThreads / kWave];
    __shared__ long long s_pre[kAppendPlanTables];  // exclusive prefix of every table's plan word
    constexpr int kSide = kQuantWaves / JW;  // jobs side by side
    __shared__ PageImage s_img[kSide];
    const long long head_old = a.flags->head_old, tail_old = a.flags->tail_old;

    // ---- the plan, in every workgroup (each thread a contiguous run of tables)
    const int per = (NT + kCommitThreads - 1) / kCommitThreads;
    const int t0 = tid * per;
    const int t1 = t0 + per < NT ? t0 + per : NT;
    // the run's first two tables stay in registers (static indices: no scratch)
    static_assert(kPlanKeep == 2, "for_tables visits two kept states");
    const TState st0 = a.tstate[min(t0, NT - 1)], st1 = a.tstate[min(t0 + 1, NT - 1)];
    auto for_tables = [&](auto&& f) {
        if (t0 < t1) f(t0, st0);
        if (t0 + 1 < t1) f(t0 + 1, st1);
        for (int t = t0 + 2; t < t1; ++t) f(t, a.tstate[t]);
    };
    long long packed = 0;
    uint32_t bits = 0;
    for_tables([&](int, const TState& s) {
        if (s.n < 0) {
            bits |= DIFFKV_ST_BAD_INPUT;
            return;
        }
        const TablePlan tp = table_plan(s, P, a.tsh);
        if (tp.held_over) bits |= DIFFKV_ST_TABLE_OVERFLOW;
        packed += plan_word(tp);
    });
    long long tot;
    uint32_t all_bits;
    const long long before = block_excl_scan<long long>(packed, s_scan, &tot, bits, s_bits, &all_bits);
    bits = all_bits & (DIFFKV_ST_BAD_INPUT | DIFFKV_ST_TABLE_OVERFLOW);
    const long long total_need = tot & 0xffffffffll;
    const int njobs = (int)(tot >> 32);
    if (bits & DIFFKV_ST_BAD_INPUT) bits = DIFFKV_ST_BAD_INPUT;
    else if (total_need > tail_old - head_old) bits |= DIFFKV_ST_OUT_OF_PAGES;
    if (bits) {  // all or nothing: no state, table or page changes
        if (blockIdx.x == 0 && tid == 0) atomicOr(a.status, bits);
        return;
    }

    // ---- workgroup 0: the state after the call -------------------------------
    if (blockIdx.x == 0) {
        for_tables([&](int t, const TState& s) {
            const TablePlan tp = table_plan(s, P, a.tsh);
#pragma unroll
            for (int sec = 0; sec < 2; ++sec) {
                a.len[2 * t + sec] = s.lold[sec] + s.cnt[sec];
                a.pages[2 * t + sec] = s.pold[sec] + tp.need[sec];
            }
        });
        for (int b = tid; b < a.B; b += kCommitThreads) a.seq_len[b] = a.sold[b] + a.new_len[b];
        if (tid == 0) a.ring_ptr[0] = head_old + total_need;
    }

    // ---- page jobs, one per wave (or workgroup) at a time -------------------------
    {
        long long pre = before;
        for_tables([&](int t, const TState& s) {
            s_pre[t] = pre;
            pre += plan_word(table_plan(s, P, a.tsh));
        });
    }
    __syncthreads();
    const int lane = lane_id();
    const int stride = (NT + kWave - 1) / kWave;
    const int side = wave_index() / JW;
    for (int job = (int)blockIdx.x * kSide + side; job < njobs; job += (int)gridDim.x * kSide) {
        // the job's table is the last whose first job is <= job (tables without
        // jobs share their successor's prefix): among every stride-th table,
        // then among the stride tables from that one on
        const int p0 = lane * stride;
        const int blk = __popcll(__builtin_amdgcn_ballot_w64(p0 < NT && (int)(s_pre[p0 < NT ? p0 : 0] >> 32) <= job)) - 1;
        const int p1 = blk * stride + lane;
        const bool in = lane < stride && p1 < NT;
        const int t = blk * stride + __popcll(__builtin_amdgcn_ballot_w64(in && (int)(s_pre[in ? p1 : 0] >> 32) <= job)) - 1;
        const TState s = uniform_state(a.tstate, t);
        JobDesc d;
        describe_job(d, t, s, table_plan(s, P, a.tsh), read_lane<long long>(s_pre[t], 0), job, P, head_old, a.tsh);
        commit_job<JW>(a, d, s_img[side]);
    }
}

// ---------------------------------------------------------------------------
// Many tables: the plan once (append_plan, one workgroup), then the jobs
// (append_commit_planned).  Every commit workgroup redoing the plan costs
// O(tables) each; past kAppendPlanTables tables one planning launch is cheaper.
// The plan writes each table's exclusive prefix, a job -> table map and the
// state after the call; a commit workgroup reads its job's table directly.
// ---------------------------------------------------------------------------
constexpr int kPlanLdsTables = 8192;  // up to this many tables the job map is built from LDS
constexpr int kMapIlp = 4;            // jobs a thread maps side by side

__global__ __launch_bounds__(kPlanThreads) void append_plan(AppendArgs a)
{
    const int tid = threadIdx.x;
    const int NT = a.B * a.Hkv;
    const int P = a.p_max;
    __shared__ long long s_scan[kPlanThreads / kWave];
    __shared__ uint32_t s_bits[kPlanThreads / kWave];
    __shared__ int32_t s_jobs[kPlanLdsTables + 1];  // first job of every table, then njobs
    const long long head_old = a.flags->head_old, tail_old = a.flags->tail_old;
    const int per = (NT + kPlanThreads - 1) / kPlanThreads;
    const int t0 = tid * per;
    const int t1 = t0 + per < NT ? t0 + per : NT;
    // the first two tables' states, loaded together and unconditionally (a
    // thread past the last table reloads table NT - 1 and ignores it)
    const TState st0 = a.tstate[min(t0, NT - 1)], st1 = a.tstate[min(t0 + 1, NT - 1)];
    auto for_tables = [&](auto&& f) {
        if (t0 < t1) f(t0, st0);
        if (t0 + 1 < t1) f(t0 + 1, st1);
        for (int t = t0 + 2; t < t1; ++t) f(t, a.tstate[t]);
    };
    long long packed = 0;
    uint32_t bits = 0;
    for_tables([&](int, const TState& s) {
        if (s.n < 0) {
            bits |= DIFFKV_ST_BAD_INPUT;
            return;
        }
        const TablePlan tp = table_plan(s, P, a.tsh);
        if (tp.held_over) bits |= DIFFKV_ST_TABLE_OVERFLOW;
        packed += plan_word(tp);
    });
    long long tot;
    uint32_t all_bits;
    const long long before = block_excl_scan<long long>(packed, s_scan, &tot, bits, s_bits, &all_bits);
    bits = all_bits & (DIFFKV_ST_BAD_INPUT | DIFFKV_ST_TABLE_OVERFLOW);
    const long long total_need = tot & 0xffffffffll;
    const int njobs = (int)(tot >> 32);
    if (bits & DIFFKV_ST_BAD_INPUT) bits = DIFFKV_ST_BAD_INPUT;
    else if (total_need > tail_old - head_old) bits |= DIFFKV_ST_OUT_OF_PAGES;
    if (njobs > a.job_cap) bits |= DIFFKV_ST_BAD_INPUT;  // never with the host's bound; keeps the map in bounds
    if (bits) {  // all or nothing: no state, table or page changes
        if (tid == 0) {
            atomicOr(a.status, bits);
            a.flags->ok = 0;
        }
        return;
    }
    const bool lds_map = NT <= kPlanLdsTables;  // job map by binary search in LDS
    long long pre = before;
    for_tables([&](int t, const TState& s) {
        const TablePlan tp = table_plan(s, P, a.tsh);
        a.tplan[t] = pre;
        const int j0 = (int)(pre >> 32);
        if (lds_map) s_jobs[t] = j0;
        else
            for (int k = 0; k < tp.jobs[0] + tp.jobs[1]; ++k) a.job_table[j0 + k] = t;
#pragma unroll
        for (int sec = 0; sec < 2; ++sec) {
            a.len[2 * t + sec] = s.lold[sec] + s.cnt[sec];
            a.pages[2 * t + sec] = s.pold[sec] + tp.need[sec];
        }
        pre += plan_word(tp);
    });
    for (int b = tid; b < a.B; b += kPlanThreads) a.seq_len[b] = a.sold[b] + a.new_len[b];
    if (tid == 0) {
        a.ring_ptr[0] = head_old + total_need;
        a.flags->njobs = njobs;
        a.flags->ok = 1;
    }
    if (lds_map) {
        // job j belongs to the last table whose first job is <= j (tables without
        // jobs share their successor's prefix); every thread maps kMapIlp jobs side
        // by side with a fixed-length search
        if (tid == 0) s_jobs[NT] = njobs;
        __syncthreads();
        int steps = 0;
        while ((1 << steps) < NT + 1) ++steps;
        for (int j0 = tid; j0 < njobs; j0 += kPlanThreads * kMapIlp) {
            int lo[kMapIlp];
#pragma unroll
            for (int i = 0; i < kMapIlp; ++i) lo[i] = 0;
            for (int st = steps - 1; st >= 0; --st) {
#pragma unroll
                for (int i = 0; i < kMapIlp; ++i) {
                    const int mid = lo[i] + (1 << st);
                    if (mid <= NT && s_jobs[mid] <= j0 + i * kPlanThreads) lo[i] = mid;
                }
            }
#pragma unroll
            for (int i = 0; i < kMapIlp; ++i)
                if (j0 + i * kPlanThreads < njobs) a.job_table[j0 + i * kPlanThreads] = lo[i];
        }
    }
}

__global__ __launch_bounds__(kCommitThreads, kCommitWaves) void append_commit_planned(AppendArgs a)
{
    __shared__ PageImage s_img[kQuantWaves];
    if (!a.flags->ok) return;
    const int njobs = a.flags->njobs;
    const long long head_old = a.flags->head_old;
    for (int job = (int)blockIdx.x * kQuantWaves + wave_index(); job < njobs; job += (int)gridDim.x * kQuantWaves) {
        const int t = __builtin_amdgcn_readfirstlane(a.job_table[job]);
        const TState s = uniform_state(a.tstate, t);
        JobDesc d;
        describe_job(d, t, s, table_plan(s, a.p_max, a.tsh), read_lane<long long>(a.tplan[t], 0), job, a.p_max, head_old, a.tsh);
        commit_job<1>(a, d, s_img[wave_index()]);
    }
}

// ---------------------------------------------------------------------------
// append_one: the whole append of a call in which every sequence takes at most
// one new token (max_new <= 1) over at most kAppendPlanTables tables -- a
// decode step -- in one launch, one workgroup per table.  One token needs no
// selection: inside the recent window it is high; in the quota form it is
// high when the high quota (clamped to the one token) is 1, else low when the
// low quota is; in the threshold form its score is compared with alpha / N as
// in append_classify.  So every workgroup derives every table's class, the
// plan (page demand, one prefix sum over tables) and the all-or-nothing
// verdict from the state before the call, then does its own table's page job
// (at most one: one token lies on one page).  No workgroup writes what another
// reads: the state after the call (lengths, pages, seq_len, ring head) is
// written by the workgroup that arrives last (arrive_count, on two levels of
// words), after every workgroup has read the state before the call.
// Workgroup 0 claims the arrival words with the call's tag as it starts
// (arrive_claim), so the arrivals, all at about the same time, count with one
// add each.
// ---------------------------------------------------------------------------
constexpr int kOnePer = (kAppendPlanTables + kCommitThreads - 1) / kCommitThreads;  // tables per thread
constexpr int kOneGroups = 16;  // first-level arrival words

inline bool append_one_call(const AppendArgs& a) { return a.max_new <= 1 && !append_planned(a.B, a.Hkv); }

__global__ __launch_bounds__(kCommitThreads) void append_one(AppendArgs a)
{
    const int tid = threadIdx.x;
    const int H = a.Hkv, B = a.B, NT = B * H, P = a.p_max;
    __shared__ long long s_scan[kCommitThreads / kWave];
    __shared__ uint32_t s_bits[kCommitThreads / kWave];
    __shared__ JobDesc s_job;
    __shared__ PageImage s_img;
    __shared__ int s_off[kAppendPlanTables];  // row offset of each sequence (new tokens of the lower ones)
    __shared__ int s_job_here, s_last;
    const unsigned long long tag = call_tag();
    if (blockIdx.x == 0 && tid <= kOneGroups)  // before any arrival, as a rule
        arrive_claim(tid < kOneGroups ? &a.flags->arrive_group[tid] : &a.flags->arrive, tag);
    const long long head_old = a.ring_ptr[0], tail_old = a.ring_ptr[1];
    if (tid == 0) s_job_here = 0;

    // ---- row offsets; each thread a run of sequences (B <= NT <= kAppendPlanTables)
    const int pb = (B + kCommitThreads - 1) / kCommitThreads;
    const int b0 = tid * pb;
    int nb[kOnePer];
    long long nsum = 0;
    uint32_t bad = 0;
#pragma unroll
    for (int i = 0; i < kOnePer; ++i) {
        nb[i] = 0;
        if (i < pb && b0 + i < B) {
            const int v = a.new_len[b0 + i];
            if (v < 0 || v > a.max_new) bad = 1;
            nb[i] = v < 0 ? 0 : (v > 1 ? 1 : v);
            nsum += nb[i];
        }
    }
    long long ntot;
    uint32_t any_bad;
    long long off = block_excl_scan<long long>(nsum, s_scan, &ntot, bad, s_bits, &any_bad);
#pragma unroll
    for (int i = 0; i < kOnePer; ++i) {
        if (i < pb && b0 + i < B) {
            s_off[b0 + i] = (int)off;
            off += nb[i];
        }
    }
    __syncthreads();
    // every count in [0, max_new] and their sum total_new: the classify
    // kernel's per-sequence row checks, taken for the whole call
    const bool bad_call = any_bad != 0 || ntot != a.total_new;

    // ---- classes and plans of every table; each thread a run of tables
    const int pt = (NT + kCommitThreads - 1) / kCommitThreads;
    const int t0 = tid * pt;
    const bool quota = a.quota != nullptr;
    TState st[kOnePer];
    long long packed = 0;
    uint32_t bits = 0;
#pragma unroll
    for (int i = 0; i < kOnePer; ++i) {
        TState& s = st[i];
        s.cnt[0] = s.cnt[1] = 0;
        s.lold[0] = s.lold[1] = s.pold[0] = s.pold[1] = 0;
        s.ring_off = 0;
        s.n = 0;
        const int t = t0 + i;
        if (i < pt && t < NT) {
            const int b = t / H, h = t - b * H;
            const int v = a.new_len[b];
            const int n = v < 0 ? 0 : (v > 1 ? 1 : v);
            s.n = n;
            s.lold[0] = a.len[2 * t];
            s.lold[1] = a.len[2 * t + 1];
            s.pold[0] = a.pages[2 * t];
            s.pold[1] = a.pages[2 * t + 1];
            if (n == 1 && !bad_call) {  // (a bad call's row offsets may lie past total_new)
                if (a.window >= 1) {
                    s.cnt[0] = 1;
                } else if (quota) {
                    const int q0 = a.quota[2 * t], q1 = a.quota[2 * t + 1];
                    const int nh = q0 < 0 ? 0 : (q0 > 1 ? 1 : q0);
                    const int nl = q1 < 0 ? 0 : (q1 > 1 - nh ? 1 - nh : q1);
                    s.cnt[0] = nh;
                    s.cnt[1] = nl;
                } else {
                    const float sc = a.score[(long long)s_off[b] * H + h];
                    const float N = (float)(a.seq_len[b] + n);
                    const float thr_h = a.alpha_h / N, thr_l = a.alpha_l / N;
                    const bool a0 = sc >= thr_h;
                    const bool a1 = a0 || sc >= thr_l;
                    s.cnt[0] = a0 ? 1 : 0;
                    s.cnt[1] = (a1 && !a0) ? 1 : 0;
                }
            }
            const TablePlan tp = table_plan(s, P, a.tsh);
            if (tp.held_over) bits |= DIFFKV_ST_TABLE_OVERFLOW;
            packed += plan_word(tp);
        }
    }
    long long tot;
    uint32_t all_bits;
    const long long before = block_excl_scan<long long>(packed, s_scan, &tot, bits, s_bits, &all_bits);
    bits = all_bits & DIFFKV_ST_TABLE_OVERFLOW;
    const long long total_need = tot & 0xffffffffll;
    if (bad_call) bits = DIFFKV_ST_BAD_INPUT;
    else if (total_need > tail_old - head_old) bits |= DIFFKV_ST_OUT_OF_PAGES;
    if (bits) {  // all or nothing: no state, table or page changes
        if (blockIdx.x == 0 && tid == 0) atomicOr(a.status, bits);
        return;
    }

    // ---- this workgroup's table: its page job, if its token is kept
    {
        long long pre = before;
#pragma unroll
        for (int i = 0; i < kOnePer; ++i) {
            const int t = t0 + i;
            if (i < pt && t < NT) {
                const TablePlan tp = table_plan(st[i], P, a.tsh);
                if (t == (int)blockIdx.x && tp.jobs[0] + tp.jobs[1] > 0) {
                    describe_job(s_job, t, st[i], tp, pre, (int)(pre >> 32), P, head_old, a.tsh);
                    const int b = t / H;
                    s_job.one = 1;
                    s_job.off_b = s_off[b];
                    s_job.sold = a.seq_len[b];
                    s_job_here = 1;
                }
                pre += plan_word(tp);
            }
        }
    }
    __syncthreads();
    if (s_job_here && wave_index() == 0) {
        JobDesc d;
        d.t = __builtin_amdgcn_readfirstlane(s_job.t);
        d.sec = __builtin_amdgcn_readfirstlane(s_job.sec);
        d.p = __builtin_amdgcn_readfirstlane(s_job.p);
        d.u0 = __builtin_amdgcn_readfirstlane(s_job.u0);
        d.u1 = __builtin_amdgcn_readfirstlane(s_job.u1);
        d.lold = __builtin_amdgcn_readfirstlane(s_job.lold);
        d.n = __builtin_amdgcn_readfirstlane(s_job.n);
        d.tslot = __builtin_amdgcn_readfirstlane(s_job.tslot);
        d.ring_idx = read_lane<long long>(s_job.ring_idx, 0);
        d.one = 1;
        d.off_b = __builtin_amdgcn_readfirstlane(s_job.off_b);
        d.sold = __builtin_amdgcn_readfirstlane(s_job.sold);
        commit_job<1>(a, d, s_img);
    }

    // ---- the workgroup arriving last writes the state after the call
    __syncthreads();
    if (tid == 0) {
        // two levels, so that no word takes more than a few dozen concurrent
        // adds: workgroup j counts in group j % kOneGroups, the last of a
        // group in the top word
        const int ng = NT < kOneGroups ? NT : kOneGroups, g = (int)blockIdx.x % kOneGroups;
        const unsigned long long gsize = NT / kOneGroups + (g < NT % kOneGroups ? 1 : 0);
        bool last = false;
        if (arrive_count(&a.flags->arrive_group[g], tag) == gsize)
            last = arrive_count(&a.flags->arrive, tag) == (unsigned long long)ng;
        s_last = last;
    }
    __syncthreads();
    if (!s_last) return;
#pragma unroll
    for (int i = 0; i < kOnePer; ++i) {
        const int t = t0 + i;
        if (i < pt && t < NT) {
            const TablePlan tp = table_plan(st[i], P, a.tsh);
#pragma unroll
            for (int sec = 0; sec < 2; ++sec) {
                a.len[2 * t + sec] = st[i].lold[sec] + st[i].cnt[sec];
                a.pages[2 * t + sec] = st[i].pold[sec] + tp.need[sec];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kOnePer; ++i)  // no other workgroup writes seq_len: this is still the length before the call
        if (i < pb && b0 + i < B) a.seq_len[b0 + i] = a.seq_len[b0 + i] + nb[i];
    if (tid == 0) a.ring_ptr[0] = head_old + total_need;
}

// ---------------------------------------------------------------------------
// Allocation alone: alloc_plan (one workgroup) + alloc_write (wave per table)
// ---------------------------------------------------------------------------
// alloc_plan is a chain of one round of loads, one prefix sum and the stores, for as
// many tables as are quickest held in registers (kAllocKeep neighbouring ones per
// thread).  Beyond those it makes a first pass over all tables for the all-or-nothing
// verdict, then rounds of one table per thread: a thread's neighbouring tables are
// strided accesses, and eight of them (8192 tables) took 16.5 us for the call where the
// rounds take 11.  4096 tables: 8.4 us, 12 with the rounds and a 64-bit sum through
// shuffles.
constexpr int kAllocKeep = 4;

template <bool KEEP>
__global__ __launch_bounds__(kPlanThreads) void alloc_plan(AllocArgs a)
{
    const int tid = threadIdx.x;
    const int NT = a.num_tables;
    __shared__ long long s_scan[kPlanThreads / kWave];
    __shared__ uint32_t s_bits[kPlanThreads / kWave];
    const long long head = a.ring_ptr[0], tail = a.ring_ptr[1];
    auto demand = [&](int t) { return make_int2(a.demand[2 * t], a.demand[2 * t + 1]); };
    auto pages = [&](int t) { return make_int2(a.pages[2 * t], a.pages[2 * t + 1]); };
    auto need = [](int2 d) { return (long long)(d.x > 0 ? d.x : 0) + (d.y > 0 ? d.y : 0); };
    auto check = [&](int2 d, int2 p) -> uint32_t {
        return (d.x < 0 || d.y < 0 ? (uint32_t)DIFFKV_ST_BAD_INPUT : 0u) |
               ((long long)p.x + p.y + d.x + d.y > a.p_max ? (uint32_t)DIFFKV_ST_TABLE_OVERFLOW : 0u);
    };
    auto place = [&](int t, int2 d, int2 p, long long off) {
        a.tstate[t] = make_int4(p.x, p.y, (int)off, d.x);
        a.pages[2 * t] = p.x + d.x;
        a.pages[2 * t + 1] = p.y + d.y;
    };
    long long sum = 0, total;
    uint32_t flags = 0, bits = 0;
    if constexpr (KEEP) {
        const int per = (NT + kPlanThreads - 1) / kPlanThreads, t0 = tid * per;
        int2 d[kAllocKeep], p[kAllocKeep];
#pragma unroll
        for (int i = 0; i < kAllocKeep; ++i) {
            if (i >= per) break;  // (uniform)
            const int t = min(t0 + i, NT - 1);
            d[i] = demand(t);
            p[i] = pages(t);
        }
#pragma unroll
        for (int i = 0; i < kAllocKeep; ++i) {
            if (i < per && t0 + i < NT) {
                sum += need(d[i]);
                flags |= check(d[i], p[i]);
            }
        }
        long long off = block_excl_scan_wide(sum, s_scan, &total, flags, s_bits, &bits);
        if (total > tail - head) bits |= DIFFKV_ST_OUT_OF_PAGES;
        if (!bits) {
#pragma unroll
            for (int i = 0; i < kAllocKeep; ++i) {
                if (i < per && t0 + i < NT) {
                    place(t0 + i, d[i], p[i], off);
                    off += d[i].x + d[i].y;
                }
            }
        }
    } else {
        for (int t = tid; t < NT; t += kPlanThreads) {
            const int2 d = demand(t);
            flags |= check(d, pages(t));
            sum += need(d);
        }
        block_excl_scan_wide(sum, s_scan, &total, flags, s_bits, &bits);
        if (total > tail - head) bits |= DIFFKV_ST_OUT_OF_PAGES;
        long long carry = 0;
        for (int t0 = 0; bits == 0 && t0 < NT; t0 += kPlanThreads) {
            const int t = t0 + tid;
            const int2 d = t < NT ? demand(t) : make_int2(0, 0);
            int all;  // (a round's pages: at most the ring's, which a 32-bit number counts)
            const int off = block_excl_scan<int>(d.x + d.y, reinterpret_cast<int*>(s_scan), &all);
            if (t < NT) place(t, d, pages(t), carry + off);
            carry += all;
        }
    }
    if (tid == 0) {
        if (bits) {
            atomicOr(a.status, bits);
            a.flags->ok = 0;
        } else {
            a.flags->head_old = head;
            a.flags->ok = 1;
            a.ring_ptr[0] = head + total;
        }
    }
}

__global__ __launch_bounds__(kWave) void alloc_write(AllocArgs a)
{
    if (!a.flags->ok) return;
    const int t = blockIdx.x;
    const int4 st = a.tstate[t];
    const int d1 = a.pages[2 * t + 1] - st.y;
    const long long base = a.flags->head_old + st.z;
    int32_t* row = a.page_table + (long long)t * a.p_max;
    for (int i = threadIdx.x; i < st.w; i += kWave) row[st.x + i] = a.ring[(base + i) % a.num_pages];
    for (int i = threadIdx.x; i < d1; i += kWave)
        row[a.p_max - 1 - (st.y + i)] = a.ring[(base + st.w + i) % a.num_pages];
}

// ---------------------------------------------------------------------------
// Compaction in two launches: compact_count (a wave per table; a workgroup
// counts a group of group_tables tables and writes the group's total) and
// compact_apply (a wave per table).  An apply wave finds its ring offset from
// the totals of the groups before its own plus the counts of the earlier
// tables of its group; groups are sized so that neither exceeds kMaxGroups
// values, i.e. one round of loads per lane, so no scan launch runs between the
// two at any table count.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool slot_live(int slot, int ph, int pl, int P)
{
    return slot < ph || slot >= P - pl;
}

constexpr int kCountWaves = 4;       // waves of a compact_count workgroup
constexpr int kCompactPlanIlp = 16;  // values a lane loads at once
constexpr int kMaxGroups = kWave * kCompactPlanIlp;

// A wave's walk over a row of P slots, the lane taking s0, s0 + 64, ...: f(s0, n)
// takes n of them with their loads in flight together (past the row's end, its
// last slot's again), one on rows that a wave covers once, else four or eight
// (rows of 2113 slots: count 12.6 -> 6.2 us, apply 20 -> 11 us).
template <typename F>
__device__ __forceinline__ void row_steps(int P, int lane, F&& f)
{
    auto walk = [&](auto n) {
        for (int s0 = lane; s0 < P; s0 += decltype(n)::value * kWave) f(s0, n);
    };
    if (P <= kWave) walk(std::integral_constant<int, 1>{});
    else if (P <= 4 * kWave) walk(std::integral_constant<int, 4>{});
    else walk(std::integral_constant<int, 8>{});
}

// ONE: one table per wave (group_tables == kCountWaves, up to kMaxGroups * kCountWaves tables)
template <bool ONE>
__global__ __launch_bounds__(kCountWaves * kWave) void compact_count(CompactArgs a)
{
    __shared__ int s_c[kCountWaves];
    const int w = wave_index();
    const int lane = threadIdx.x & (kWave - 1);
    const int P = a.p_max;
    const int GT = ONE ? kCountWaves : a.group_tables;
    const int t0 = blockIdx.x * GT;
    const int t1 = ONE ? min(a.num_tables, t0 + w + 1) : min(a.num_tables, t0 + GT);
    int gsum = 0;
    for (int t = t0 + w; t < t1; t += kCountWaves) {
        int ph = a.pages[2 * t], pl = a.pages[2 * t + 1];
        ph = ph < 0 ? 0 : (ph > P ? P : ph);
        pl = pl < 0 ? 0 : (pl > P - ph ? P - ph : pl);
        const uint8_t* rel = a.release + (long long)t * P;
        int c = 0;
        row_steps(P, lane, [&](int s0, auto ilp) {
            constexpr int N = decltype(ilp)::value;
            uint8_t r[N];
#pragma unroll
            for (int i = 0; i < N; ++i) r[i] = rel[min(s0 + i * kWave, P - 1)];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int s = s0 + i * kWave;
                c += (s < P && r[i] != 0 && slot_live(s, ph, pl, P));
            }
        });
        c = wave_isum_w<kWave>(c);
        if (lane == 0) a.count[t] = c;
        gsum += c;
    }
    if (lane == 0) s_c[w] = gsum;
    __syncthreads();
    if (threadIdx.x == 0) {
        int g = 0;
#pragma unroll
        for (int i = 0; i < kCountWaves; ++i) g += s_c[i];
        a.offset[blockIdx.x] = g;  // the group's total
        // the end pointer before the call
        if (blockIdx.x == 0) a.flags->tail_old = a.ring_ptr[1];
    }
}

// sum of v[0 .. n) and of v[0 .. below) over the wave, n <= kMaxGroups: all
// loads in flight together (unconditional, clamped to the last element)
__device__ __forceinline__ void wave_sum_prefix(const int32_t* v, int n, int below, int lane, int& tot, int& pre)
{
    int cv[kCompactPlanIlp];
#pragma unroll
    for (int k = 0; k < kCompactPlanIlp; ++k) cv[k] = v[min(lane + k * kWave, n - 1)];
#pragma unroll
    for (int k = 0; k < kCompactPlanIlp; ++k) {
        const int i = lane + k * kWave;
        const int c = i < n ? cv[k] : 0;
        tot += c;
        pre += i < below ? c : 0;
    }
}

// One wave per table; the live part of the row is staged in LDS (dynamic
// shared memory of 2*p_max ints) with each slot's release flag in the sign bit
// of its page ID (IDs are non-negative), so the squeeze writes in place and no
// global load sits between the ring stores (a byte load may alias them, so the
// compiler would keep each after the last store).  The wave of table 0
// advances the end pointer by the call's total.
template <bool ONE>
__global__ __launch_bounds__(kWave) void compact_apply(CompactArgs a)
{
    extern __shared__ int32_t s_row[];  // [0, P): old IDs (sign bit: released), [P, 2P): new row
    const int t = blockIdx.x;
    const int lane = threadIdx.x;
    const int NT = a.num_tables;
    const int P = a.p_max;
    int ph = a.pages[2 * t], pl = a.pages[2 * t + 1];
    const int len0 = a.len[2 * t], len1 = a.len[2 * t + 1];
    const long long tail_old = a.flags->tail_old;
    const int GT = ONE ? kCountWaves : a.group_tables;
    const int ng = (NT + GT - 1) / GT, g = t / GT, t0 = g * GT;
    int tot = 0, before = 0;
    wave_sum_prefix(a.offset, ng, g, lane, tot, before);  // the groups before g
    if (ONE) {
        if (lane < t - t0) before += a.count[t0 + lane];  // its group's tables before t
    } else {
        for (int i = t0 + lane; i < t; i += kWave) before += a.count[i];
    }
    ph = ph < 0 ? 0 : (ph > P ? P : ph);  // same clamp as compact_count
    pl = pl < 0 ? 0 : (pl > P - ph ? P - ph : pl);
    const int T0 = a.T[0], T1 = a.T[1];
    const uint8_t* rel = a.release + (long long)t * P;
    int32_t* row = a.page_table + (long long)t * P;
    int32_t* s_new = s_row + P;
    // the whole row, without waiting for the page counts: every load of the
    // wave is then in flight at once (slots outside the sections are not read)
    row_steps(P, lane, [&](int s0, auto ilp) {
        constexpr int N = decltype(ilp)::value;
        int32_t id[N];
        uint8_t r[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int s = min(s0 + i * kWave, P - 1);
            id[i] = row[s];
            r[i] = rel[s];
        }
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (s0 + i * kWave < P) s_row[s0 + i * kWave] = id[i] | (r[i] != 0 ? (int32_t)0x80000000 : 0);
    });
    tot = wave_isum_w<kWave>(tot);
    const int my_off = wave_isum_w<kWave>(before);
    if (t == 0 && lane == 0) a.ring_ptr[1] = tail_old + tot;
    const long long n = a.num_pages;
    // ring position of this table's first released ID, reduced once; later
    // positions pass n at most once (rank < released slots <= pages in the pool)
    const long long start = (tail_old % n + my_off) % n;
    const uint64_t below = (1ull << lane) - 1ull;
    __syncthreads();
    auto ring_at = [&](int k) -> int32_t& {
        long long i = start + k;
        i = i >= n ? i - n : i;
        return a.ring[i];
    };
    // released IDs to the ring in ascending slot order; kept high IDs packed left
    int rank = 0, hi_keep = 0, drop0 = 0, drop1 = 0;
    for (int c = 0; c < ph; c += kWave) {
        const int s = c + lane;
        const bool live = s < ph;
        const int32_t id = live ? s_row[s] : 0;
        const bool r = live && id < 0;
        const uint64_t mr = __ballot(r);
        const uint64_t mk = __ballot(live && !r);
        if (r) {
            ring_at(rank + __popcll(mr & below)) = id & 0x7fffffff;
            int f = len0 - s * T0;
            drop0 += f < 0 ? 0 : (f > T0 ? T0 : f);
        }
        if (live && !r) s_new[hi_keep + __popcll(mk & below)] = id;
        rank += __popcll(mr);
        hi_keep += __popcll(mk);
    }
    for (int c = P - pl; c < P; c += kWave) {
        const int s = c + lane;
        const int32_t id = s < P ? s_row[s] : 0;
        const bool r = s < P && id < 0;
        const uint64_t mr = __ballot(r);
        if (r) {
            ring_at(rank + __popcll(mr & below)) = id & 0x7fffffff;
            int f = len1 - (P - 1 - s) * T1;
            drop1 += f < 0 ? 0 : (f > T1 ? T1 : f);
        }
        rank += __popcll(mr);
    }
    // kept low IDs packed right, in section order (section page k sits at slot P-1-k)
    int lo_keep = 0;
    for (int c = 0; c < pl; c += kWave) {
        const int k = c + lane;
        const int s = P - 1 - k;
        const int32_t id = k < pl ? s_row[s] : -1;
        const bool keep = k < pl && id >= 0;
        const uint64_t mk = __ballot(keep);
        if (keep) s_new[P - 1 - (lo_keep + __popcll(mk & below))] = id;
        lo_keep += __popcll(mk);
    }
    __syncthreads();
    for (int s = lane; s < ph; s += kWave) row[s] = s < hi_keep ? s_new[s] : -1;
    for (int s = P - pl + lane; s < P; s += kWave) row[s] = s >= P - lo_keep ? s_new[s] : -1;
    drop0 = wave_isum_w<kWave>(drop0);
    drop1 = wave_isum_w<kWave>(drop1);
    if (lane == 0) {
        a.pages[2 * t] = hi_keep;
        a.pages[2 * t + 1] = lo_keep;
        a.len[2 * t] = len0 - drop0;
        a.len[2 * t + 1] = len1 - drop1;
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_append(const AppendArgs& args, int grid_quant, hipStream_t st)
{
    AppendArgs a = args;
    if (append_one_call(a)) return launch1(append_one, (unsigned)(a.Hkv * a.B), kCommitThreads, st, a);
    // a table's tiles go to several workgroups while all of these stay within kClsBusyGroups
    // (up to half as many tables)
    const int tables = a.Hkv * a.B, tiles = (int)(((long long)a.max_new + kClsTile - 1) / kClsTile);
    const int room = kClsBusyGroups / tables;
    a.cls_split = tiles < room ? tiles : room;
    if (a.cls_split < 1) a.cls_split = 1;
    hipError_t e = launch1(a.max_new <= kClsThreads ? append_classify<1> : append_classify<kClsPer>,
                           (unsigned)(tables * a.cls_split), kClsThreads, st, a);
    if (e != hipSuccess) return e;
    if (append_planned(a.B, a.Hkv)) {
        e = launch1(append_plan, 1, kPlanThreads, st, a);
        if (e != hipSuccess) return e;
        return launch1(append_commit_planned, (unsigned)grid_quant, kCommitThreads, st, a);
    }
    if (a.job_cap <= (a.max_new < kCommitFewTokens ? 1 : 2) * kCommitFewJobs)
        return launch1(append_commit<kQuantWaves>, (unsigned)max(a.job_cap, 1), kCommitThreads, st, a);
    return launch1(append_commit<1>, (unsigned)grid_quant, kCommitThreads, st, a);
}

hipError_t launch_alloc(const AllocArgs& a, hipStream_t st)
{
    hipError_t e = launch1(a.num_tables <= kAllocKeep * kPlanThreads ? alloc_plan<true> : alloc_plan<false>, 1, kPlanThreads,
                           st, a);
    if (e != hipSuccess || a.num_tables == 0) return e;
    return launch1(alloc_write, (unsigned)a.num_tables, kWave, st, a);
}

hipError_t launch_compact(const CompactArgs& args, hipStream_t st)
{
    if (args.num_tables == 0) return hipSuccess;
    CompactArgs a = args;
    // tables per count group: at least one per wave, and few enough groups that an
    // apply wave sums them (and its group's earlier counts) in one round of loads
    const long long per = ((long long)a.num_tables + kMaxGroups - 1) / kMaxGroups;
    a.group_tables = (int)(per < kCountWaves ? kCountWaves : per);
    if (a.group_tables > kMaxGroups) return hipErrorInvalidValue;
    const size_t lds = (size_t)2 * a.p_max * sizeof(int32_t);
    const unsigned groups = (unsigned)((a.num_tables + a.group_tables - 1) / a.group_tables);
    const bool one = a.group_tables == kCountWaves;
    hipError_t e = one ? launch1(compact_count<true>, groups, kCountWaves * kWave, st, a)
                       : launch1(compact_count<false>, groups, kCountWaves * kWave, st, a);
    if (e != hipSuccess) return e;
    return one ? launch1(compact_apply<true>, (unsigned)a.num_tables, kWave, st, a, lds)
               : launch1(compact_apply<false>, (unsigned)a.num_tables, kWave, st, a, lds);
}

}  // namespace dkv
