// internal.hpp -- argument blocks and launchers shared by the API and kernels.
#pragma once

#include "common.hpp"

namespace dkv {

struct TState {        // per-table scratch of one append call
    int32_t cnt[2];    // kept new tokens per section
    int32_t lold[2];   // section lengths before the call
    int32_t pold[2];   // pages held before the call
    int32_t ring_off;  // first ring index of this table's new pages, from head_old
    int32_t n;         // new tokens of the table's sequence
};

struct LayoutArgs {
    int p_max;
    int T[2];
    int kb[2], vb[2];  // key and value bits per section
    int tsh;           // log2 of the tokens per page: high section in bits 0-7, low in 8-15
    long long page_bytes;
    int off_kcode[2], off_kmeta[2], off_vcode[2], off_vmeta[2], off_score[2], off_pos[2];
};

struct AppendArgs : LayoutArgs {
    uint8_t* pool;
    long long num_pages;
    int32_t* page_table;
    int32_t* pages;
    int32_t* len;
    int32_t* seq_len;
    int32_t* ring;
    int64_t* ring_ptr;
    uint32_t* status;
    int B, Hkv;
    long long total_new;
    int max_new;
    const int32_t* new_len;
    const uint16_t* k;
    const uint16_t* v;
    const float* score;
    const int32_t* quota;
    float alpha_h, alpha_l;
    int window;
    CallFlags* flags;
    TState* tstate;
    int32_t* sold;
    int32_t* row_off;
    int32_t* ord;
    long long* tplan;    // [tables] exclusive prefix (new pages | jobs << 32), planned path
    int32_t* job_table;  // [job_cap] table of each page job, planned path
    int job_cap;
    int cls_split;       // classify workgroups per table
};

// Above this many tables an append plans once in its own launch instead of in
// every commit workgroup.
constexpr int kAppendPlanTables = 1024;
constexpr int kAppendJobsPerGroup = 4;  // page jobs a commit workgroup runs side by side (one per wave)
inline bool append_planned(long long B, long long Hkv) { return B * Hkv > kAppendPlanTables; }

struct AllocArgs {
    int p_max;
    long long num_pages;
    int32_t* page_table;
    int32_t* pages;
    int32_t* ring;
    int64_t* ring_ptr;
    uint32_t* status;
    int num_tables;
    const int32_t* demand;
    CallFlags* flags;
    int4* tstate;  // {pages_hi_old, pages_lo_old, ring_off, demand_hi}
};

struct CompactArgs {
    int p_max;
    int T[2];
    long long num_pages;
    int32_t* page_table;
    int32_t* pages;
    int32_t* len;
    int32_t* ring;
    int64_t* ring_ptr;
    int num_tables;
    const uint8_t* release;
    CallFlags* flags;
    int32_t* count;    // [num_tables] released live slots of each table
    int32_t* offset;   // [groups] released slots of each group of group_tables tables
    int group_tables;  // tables per compact_count workgroup
};

// per-table decision of one generation step
enum GenAction : int32_t {
    kGenNone = 0,
    kGenHighVictimToLow = 1,  // candidate stays high; the high victim moves to the low section
    kGenHighVictimOut = 2,    // candidate stays high; the high victim is removed
    kGenCandToLow = 3,        // the candidate moves to the low section
    kGenCandOut = 4           // the candidate is removed
};

struct GenArgs : LayoutArgs {
    uint8_t* pool;
    long long num_pages;
    int32_t* page_table;
    int32_t* pages;
    int32_t* len;
    const int32_t* seq_len;
    int32_t* ring;
    int64_t* ring_ptr;
    uint32_t* status;
    int Hkv, num_tables;
    float alpha_h, alpha_l;
    int window;
    CallFlags* flags;  // ring head/tail before the call; `ok` of the separate plan kernel
    int4* act;         // [num_tables] {action, high index leaving, low index written, 0}
    int4* ids;         // [num_tables] page IDs {leaving token, last high token, low target or -1, 0}
    int32_t* demand;   // [num_tables] bit 0: takes a low page; bit 1: would exceed p_max
    int32_t* offset;   // [num_tables] ring offset of the table's page (separate plan kernel)
};

struct AttnArgs {
    int p_max;
    long long page_bytes;
    long long num_pages;
    int off_kcode[2], off_kmeta[2], off_vcode[2], off_vmeta[2];
    const uint8_t* pool;
    const int32_t* page_table;
    const int32_t* len;
    int B, Hkv, Hq;
    const uint16_t* q;
    float scale_log2;    // sm_scale * log2(e)
    float* out;
    float* lse;
    int splits;          // 0: balanced shares; S >= 1: min(S, pages) ranges per table
    unsigned long long* arrive;  // [T] arrival words of split tables (call tag, count)
    float* part;         // partial states {max, sum, acc[kD]} per head
    int layout;          // index into kLayoutFmts
};

// most shares of the balanced attention mode (sizes its workspace)
constexpr int kAttnMaxWorkers = 2048;

hipError_t launch_append(const AppendArgs& a, int grid_quant, hipStream_t st);
hipError_t launch_alloc(const AllocArgs& a, hipStream_t st);
hipError_t launch_compact(const CompactArgs& a, hipStream_t st);
hipError_t launch_generation(const GenArgs& g, hipStream_t st);
hipError_t launch_attention(AttnArgs a, hipStream_t st);

// Significance update of one decode step: every kept token's score in its page
// becomes the running mean of the softmax probabilities it has received (max
// over the KV head's query heads), from the logits of q and the lse that the
// attention call with the same q wrote.
struct SigArgs {
    int p_max;
    long long num_pages;
    int off_score[2], off_pos[2];
    uint8_t* pool;
    const int32_t* page_table;
    const int32_t* len;
    const int32_t* seq_len;
    int B, Hkv, Hq;
    const uint16_t* q;
    float scale_log2;
    const float* lse;   // [B][Hq] natural log, from the attention call
    int layout;         // index into kLayoutFmts
    int shares;         // workgroups per table
};
hipError_t launch_significance(const SigArgs& a, hipStream_t st);
// The mode an attention call with `splits` runs in on the current device:
// S >= 1 page ranges per table (S = 1: no split) or -1 (balanced shares);
// *workers = the balanced mode's share count.
hipError_t attention_mode(int gq, int li, long long T, int splits, int* mode, int* workers);

// Prompt-phase significance: rows of q [total_new][Hq][kD] and k
// [total_new][Hkv][kD] concatenated per sequence; score [total_new][Hkv].
struct PromptArgs {
    int B, Hq, Hkv, max_new;
    long long total_new;
    const int32_t* new_len;
    const uint16_t* q;
    const uint16_t* k;
    const float* lse;    // [total_new][Hq] natural log from the caller, or null: the row pass computes it
    float scale_log2;    // sm_scale * log2(e)
    float* score;
    long long* off;      // [B] first row of each sequence (workspace)
    int32_t* nlen;       // [B] rows of each sequence, clamped to max_new and total_new (workspace)
    float* lse2;         // [total_new][Hq] row log2-sum-exp (workspace)
    int* ctr;            // [2][kPromptQueues] work counters of the two passes, kPromptCtrStride apart (workspace)
    int* start;          // [2][kPromptQueues][groups + 1] first items (workspace)
    int groups;          // groups of pairs per list
    int once[2];         // the passes with one workgroup per item
    int row_pos, row_groups;  // the row pass's positions per block and head groups
    int segs;            // query segments per key block of the column pass
    float* part;         // [segs][total_new][Hkv] the segments' sums, segs > 1 (workspace)
};

// Lists of work items (one per XCD), pairs per group of a list, ints between two counters
// (a cache line each: sixteen in one line took 60 us to find empty).
constexpr int kPromptQueues = 8;
constexpr int kPromptGroup = 8;
constexpr int kPromptCtrStride = 32;

// Query segments per 256-key block of the column pass: where there are fewer key
// blocks than would keep the device busy, each block's queries are cut, down to
// eight ways (the first block of one 4999-token prompt holds an eightieth of the
// work of its 160 blocks, so the pass took as long as that one block: 867 us at 64
// query heads, 210 us cut).  A sum over segments replaces the direct store.  The numbers
// of blocks are for a device of 256 CUs, two workgroups each.
constexpr int kPromptBusyBlocks = 2048;
constexpr int kPromptMaxSegs = 8;
constexpr int kPromptFewStagesBlocks = 512;

// Most values the segments' sums take for any number of KV heads (Hq / 8 .. Hq):
// the workspace size is not told it.
inline long long prompt_part_rows(long long B, long long Hq, long long total_new)
{
    const long long per_head = total_new / 256 + B;
    if (per_head <= 0 || per_head * ((Hq + 7) / 8) >= kPromptBusyBlocks) return 0;
    const long long cut = kPromptBusyBlocks / per_head + 1 + Hq, all = kPromptMaxSegs * Hq;
    return total_new * (cut < all ? cut : all);
}

// No more segments than the longest prompt has stages of query positions (128 at one query head
// per KV head, 64 at two, else 32), and for prompts of a few stages only as many as
// run at once: a stage is then worth less than the launch that adds the segments (256
// prompts of 100 tokens, 4 / 1 heads: 21.0 us in four segments, 17.6 whole).
inline int prompt_segs(long long B, long long Hq, long long Hkv, long long total_new, long long max_new)
{
    const long long blocks = (total_new / 256 + B) * Hkv;
    if (blocks <= 0) return 1;
    long long s = (kPromptBusyBlocks + blocks - 1) / blocks;
    if (s > kPromptMaxSegs) s = kPromptMaxSegs;
    const long long g = Hq / Hkv, stage = g == 1 ? 128 : (g == 2 ? 64 : 32), stages = (max_new + stage - 1) / stage;
    if (s > stages) s = stages;
    if (stages <= kPromptMaxSegs && s > kPromptFewStagesBlocks / blocks) s = kPromptFewStagesBlocks / blocks;
    // (never more than the workspace holds, whatever the constants above)
    const long long room = total_new > 0 ? prompt_part_rows(B, Hq, total_new) / (total_new * Hkv) : 1;
    if (s > room) s = room;
    return (int)(s < 1 ? 1 : s);
}
hipError_t launch_prompt_significance(const PromptArgs& a, int g, hipStream_t st);

// Fixed device scratch of diffkv_decode_attention_noalloc, one per device.
constexpr long long kNoAllocScratchBytes = 8ll << 20;
hipError_t noalloc_scratch(void** ptr);

}  // namespace dkv
