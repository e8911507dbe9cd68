// pj_internal.h -- types and kernel launchers shared by the device and host parts of libpassjoin.
//
// Device data layout (all in HBM, built once per string set):
//   * length-sorted arena: strings reordered by (length, id) and stored back to back, each at a
//     16-byte aligned slot of stride(l) = round_up(l, 16) bytes, so the byte offset of the string at
//     sorted position g of length l is gbase[l] + (g - lenstart[l]) * stride(l) -- computed from
//     two per-length tables, never gathered per string;
//   * perm[g] = original id of sorted position g, slen[g] = its length;
//   * segment index for one tau: (key, g) entries sorted by key, key = group(l, i) << 40 | code,
//     group(l, i) = (l - (tau+1)) * (tau+1) + (i-1), code = the segment's packed symbol codes
//     when they fit 40 bits (exact), or 40 bits of its polynomial hash, either spread by a
//     multiplication; equal keys form one inverted list L_l^i(w) whose members are in ascending g
//     (Sec. 3.2);
//   * list records {key, start, count} in key order, and a directory into them by (l, i) group and
//     leading code bits.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pj {

constexpr int kLenMax = 2047;          // PJ_LEN_MAX
constexpr int kLenTab = kLenMax + 2;   // per-length tables are indexed 0 .. kLenMax + 1
constexpr int kTauMax = 63;            // PJ_TAU_MAX
constexpr int kHashBits = 40;          // hash bits kept in an index key

__host__ __device__ inline int64_t stride_of(int l) { return (int64_t)((l + 15) & ~15); }
constexpr int kBatchedRoundsMax = 16;   // rounds of 64 candidates per batched-verify wave chunk
constexpr int kInlineMaxLen = 64;       // longest string the list-segment kernel keeps in registers

// Length classes of the big lists in the batched path (strings of at most kLenClass0 bytes, at
// most kLenClass1, longer): each class is verified by the list-segment kernel whose lane slots
// its strings fit (a class split at 48 bytes measured no faster).  The small lists are split
// the same way, for the batched kernel's LDS-staged form.  Hit buckets: small lists by class
// and slot, then big lists by class and slot.
constexpr int kLenClasses = 3;
constexpr int kLenClass0 = 40, kLenClass1 = 64;
constexpr int kHitBuckets = 128 * kLenClasses;
__host__ __device__ inline int len_class(int l)
{
    return (l > kLenClass0 ? 1 : 0) + (l > kLenClass1 ? 1 : 0);
}
// longest indexed string of length class c in a set whose longest string has ymax bytes
inline int class_maxlen(int c, int ymax)
{
    const int cap = c == 0 ? kLenClass0 : c == 1 ? kLenClass1 : ymax;
    return ymax < cap ? ymax : cap;
}

// Symbol map of an indexed set: code[b] = 1 + rank of byte b among the bytes the set contains
// (0: absent), bits = bit length of the largest code.  A segment of at most exact_len =
// floor(kHashBits / bits) bytes is keyed by its packed codes (exact: no byte guard); a longer
// one by a hash of its bytes.  A probe segment with an absent byte packs a 0 code, which no
// indexed key has.
struct SymMap {
    const uint16_t* code = nullptr;   // device [256]
    int bits = 9;
    int exact_len = kHashBits / 9;
};

// Length-sorted device arena of one string set.
struct DevSet {
    int64_t n = 0;
    int lmin = 0, lmax = -1;            // smallest / largest length present (lmax < lmin: empty)
    int64_t arena_bytes = 0;
    uint8_t* sarena = nullptr;          // padded, length-sorted bytes
    int32_t* perm = nullptr;            // [n] sorted position -> id
    uint16_t* slen = nullptr;           // [n] sorted position -> length
    // sets to be indexed: the bytes present (bitmap of 8 words, scratch) and their symbol codes,
    // which the first index writes
    uint32_t* bitmap = nullptr;
    uint16_t* code = nullptr;
    int32_t* lenstart = nullptr;        // [kLenTab + 1] first sorted position of each length
    int64_t* gbase = nullptr;           // [kLenTab] byte base of each length group
    // host copies of the per-length tables
    int32_t h_lenstart[kLenTab + 1];
    int64_t h_gbase[kLenTab];
};

// Segment index of one set for one tau.
struct DevIndex {
    int tau = 0;
    SymMap sym;
    int64_t entries = 0;                // (string, slot) entries
    int64_t lists = 0;                  // distinct keys (inverted lists)
    uint32_t* vals = nullptr;           // [entries] sorted position g of the string
    // the lists' records {key lo, key hi, start, count} in key order, closed by one of the
    // largest key; the directory into them: group g = key >> 40 owns the entries
    // [gdir[g], gdir[g + 1]) of dir, each {bit map, first record} (pj_device_common.h)
    uint4* recs = nullptr;              // [lists + 1]
    uint2* dir = nullptr;
    uint32_t* gdir = nullptr;           // [(lmax - tau) * (tau + 1) + 1]
    // inline copies of the members' strings in index order (strings of at most kInlineMaxLen
    // bytes; nullptr otherwise): entry j of length l at inl + inl_base[l] + j * stride_of(l)
    uint8_t* inl = nullptr;
    int64_t* inl_base = nullptr;        // [kLenTab] device
    // shared-prefix verification (Sec. 5.3): every list's members in content order (sorted by
    // the first 8 bytes of the string, then g), at the list's positions; and the full length of
    // each list at its first entry (other entries unused).  nullptr when not built.
    uint32_t* svals = nullptr;          // [entries]
    uint32_t* runlen = nullptr;         // [entries]
};

// Per-threshold view of a multi-tau index (serving): the records, directory and list entries of
// the index built for tau, and the divisor for tau+1.  Indexed by tau.
struct IndexRef {
    const uint4* recs;
    const uint32_t* vals;
    const uint2* dir;
    const uint32_t* gdir;
    uint32_t div_m;     // ceil(2^21 / (tau + 1)), see Div
    uint32_t present;   // 1 if an index for this tau exists
};

// One selected substring that found a non-empty list: candidates (vals[start + m], x, i, p).
struct Hit {
    uint32_t gx;      // sorted position of the probe string in the probe set
    uint32_t start;   // first entry of the list in DevIndex::vals
    uint32_t count;   // list members that are candidates (after the visiting-order filter)
    uint32_t meta;    // (p - 1) | (i - 1) << 11 | l << 17
};

struct ProbeParams {
    // probe side
    const uint8_t* x_arena; const uint16_t* x_slen; const int32_t* x_lenstart;
    const int64_t* x_gbase;
    uint32_t g_begin;           // first probe position
    uint64_t threads;           // probe positions * nl * (tau+1)
    int nl;                     // lengths probed per string: tau+1 (self) or 2tau+1 (two sets)
    int self;                   // 1: self-join (l in [n-tau, n], y before x when l == n)
    const int32_t* q_tau;       // per-probe tau by sorted position (mixed-tau batch) or nullptr
    const IndexRef* refs;       // [kTauMax + 1] when q_tau is set
    // index side
    const int32_t* y_lenstart;  // to know which lengths are present
    const uint32_t* vals; const uint4* recs; const uint2* dir; const uint32_t* gdir;
    int tau;                    // uniform tau, or the largest tau of a mixed batch
    int ymin, ymax;             // indexed lengths present
    // output
    Hit* hits; uint64_t hit_cap;
    unsigned long long* counters;   // [0] hits, [1] candidates, [2] selected
    int shards;                     // statistics lines after them (0: none)
    // device-resident probe count (captured batches): threads = *nx_dev * nl * (tau + 1)
    const uint32_t* nx_dev;
    SymMap sym;                 // the indexed set's symbol map (keys)
    int selection;              // PJ_SELECT_* window of start positions
    // the (length, slot) pairs of a probe string in the order the threads take them: a
    // permutation of 0 .. nl * (tau+1) - 1 grouped by window size, so that a wave's lanes walk
    // windows of one size (launch_probe_order); nullptr: natural order
    const uint16_t* order;
};

// Tiles of the pair-major probe: up to 64 consecutive probe strings of one length of at most
// kTileMaxLen bytes; first[l] = the first tile of length l (of the lengths of one launch).
constexpr int kTileMaxLen = 127;
struct ProbeTiles {
    uint32_t first[kTileMaxLen + 1];
    uint32_t tiles;
    uint32_t groups;            // a tile's (length, slot) pairs are split over this many waves
    int maxlen;                 // longest probe string of a tile
};

// Multi-match window positions of a probe string as a list, for the probe of long strings: item
// r << 8 | s is position s of the (unclipped) window of pair r = dl * (tau+1) + (i-1), in the order
// of r.  Pairs are taken kItemPairs at a time; their items are items[chunk[c] .. chunk[c + 1]).
constexpr int kItemPairs = 512;
constexpr int kItemChunks = ((2 * kTauMax + 1) * (kTauMax + 1) + kItemPairs - 1) / kItemPairs;
struct ProbeItems {
    const uint32_t* items;
    const uint32_t* chunk;      // [chunks + 1]
    int chunks;
};

struct VerifyParams {
    const uint8_t* x_arena; const uint16_t* x_slen; const int32_t* x_lenstart;
    const int64_t* x_gbase;
    const uint8_t* y_arena; const int32_t* y_lenstart; const int64_t* y_gbase;
    const uint32_t* vals;
    // inline member strings of the index (DevIndex::inl / inl_base), or nullptr
    const uint8_t* y_inl; const int64_t* y_inl_base;
    const Hit* hits; const unsigned long long* prefix;   // [nhits + 1] exclusive prefix of counts
    uint64_t nhits; uint64_t ncand;
    int tau;                                              // uniform tau or the batch's largest
    int y_maxlen;                                         // longest indexed string
    const int32_t* q_tau;                                 // per-probe tau or nullptr
    const IndexRef* refs;                                 // [kTauMax + 1] when q_tau is set
    uint64_t* out; uint64_t out_cap;                      // accepted (gx << 32 | gy)
    unsigned long long* counters;    // [3] accepted, [4] cells, [5] guard misses, [7] list-segment cells
    int shards;                      // statistics lines after them (0: none)
    // device-resident sizes (captured batches): [0] hits, [1] candidates, [2] wave chunks, [4]
    // rounds per chunk; when set they replace nhits, ncand, the launch's chunk count, wave_rounds
    const unsigned long long* dev_counts;
    int exact_len;              // segments up to this length have exact keys (no byte guard)
    int wave_rounds;            // batched verification: rounds of 64 candidates per wave chunk
    // shared-prefix verification: content-ordered lists and list lengths (DevIndex::svals,
    // runlen), and whether this is a self-join (lists of the probe's own length are then
    // filtered to the members visited before it, member by member)
    const uint32_t* svals;
    const uint32_t* runlen;
    int self;
};
// Join counters: a line of kCounterLine words ([0] hits, [3] accepted: positions that blocks
// reserve), then kStatShards lines of statistics in the same places, which the host adds up.  Words
// 10 + c of the first kTicketLines of these are the chunk tickets of length class c's list kernel.
// [8] rows and [9] cells that shared-prefix verification took from an earlier member's DP instead
// of computing them.
constexpr int kCounterLine = 16, kStatShards = 32;
constexpr int kTicketWord = 10, kTicketLines = 8;
constexpr int kJoinCounters = kCounterLine * (1 + kStatShards);

// ---- launchers (pj_device.hip) ----
// lcount: kLenTab + 1 zeroed words: strings per length, errors found (1 first offset not 0, 2 offsets
// decrease, 4 a string too long); also writes lenstart [kLenTab + 1] and gbase [kLenTab],
// and clears bitmap [8] and code [256] (both or neither nullptr)
hipError_t launch_length_hist(const int32_t* offs, int64_t n, int32_t* lcount, int32_t* lenstart,
                              int64_t* gbase, uint32_t* bitmap, uint16_t* code, hipStream_t s);
hipError_t launch_iota_len_keys(const int32_t* offs, int64_t n, uint32_t* keys, uint32_t* vals,
                                hipStream_t s);
hipError_t launch_pack_arena(const uint8_t* bytes, const int32_t* offs, const int32_t* perm,
                             int64_t n, const int32_t* lenstart, const int64_t* gbase,
                             uint8_t* sarena, uint16_t* slen, int lmax, uint32_t* bitmap,
                             hipStream_t s);   // bitmap: 8 zeroed words for the bytes present, or null
// stable sort of the ids by length (strings of at most 255 bytes; hist: strings per length)
hipError_t launch_length_sort(const int32_t* offs, int64_t n, const int32_t* hist, int32_t* perm,
                              void* tmp, size_t tmp_bytes, hipStream_t s);
hipError_t launch_emit_segments(const DevSet& S, int tau, int64_t g_first, int64_t g_count,
                                int64_t* inl_base, uint64_t* keys, uint32_t* vals, hipStream_t s);
hipError_t launch_gather_inline(const DevSet& S, const uint64_t* keys, const uint32_t* vals,
                                int64_t E, int tau, const int64_t* inl_base, uint8_t* inl,
                                hipStream_t s);
// the lists' records and directory: recs[0 .. nruns], gdir[0 .. ngroups] and the entries of dir
// (at most nruns + ngroups, zeroed by the caller); bounds: 2 * ngroups words of scratch (zeroed by
// the caller), words: ngroups
hipError_t launch_list_dir(const uint64_t* keys, const uint32_t* runstart, uint32_t nruns, uint32_t E,
                           uint32_t ngroups, uint32_t* bounds, uint32_t* words, void* scan_tmp,
                           size_t scan_bytes, uint4* recs, uint32_t* gdir, uint2* dir,
                           hipStream_t s);
hipError_t launch_probe(const ProbeParams& P, int max_blocks, hipStream_t s);
// pair-major probe of the strings of T's tiles, and multi-match probe of the strings
// g_first .. g_end - 1 (of at most maxlen bytes), a block each; uniform tau
hipError_t launch_probe_tiles(const ProbeParams& P, const ProbeTiles& T, int max_blocks,
                              hipStream_t s);
hipError_t launch_probe_long(const ProbeParams& P, const ProbeItems& I, uint32_t g_first,
                             uint32_t g_end, int maxlen, int max_blocks, hipStream_t s);
// the item list of a (tau, nl): items has room for probe_item_count entries, chunk for
// kItemChunks + 1
uint64_t probe_item_count(int tau, int nl, int self);
hipError_t launch_probe_items(int tau, int nl, int self, uint32_t* items, uint32_t* chunk,
                              hipStream_t s);
// order[0 .. nl * (tau+1)): the (length, slot) pairs r = dl * (tau+1) + (i-1) of a probe string
// by decreasing multi-match window size (any order within a size)
hipError_t launch_probe_order(int tau, int nl, int self, uint16_t* order, hipStream_t s);
hipError_t launch_hit_counts(const Hit* hits, uint64_t nh, uint32_t* counts, hipStream_t s);
hipError_t launch_verify(const VerifyParams& V, int grid, hipStream_t s);
// batched path: bucket the hits (small lists, then big ones, each by length class and then
// slot) into out, bucket regions in order; bb: kHitBuckets * slot_bucket_grid(nh_cap) u32,
// bb_off: one more (bb_off[64 * c * grid] = first hit of the small lists of length class c,
// bb_off[64 * (kLenClasses + c) * grid] that of the big lists), scan_tmp:
// scan_tmp_bytes(kHitBuckets * grid).  Then verify with per-wave chunks
// (first: batched_chunks(ncand) u32 of scratch)
unsigned slot_bucket_grid(uint64_t nh_cap);
hipError_t launch_slot_bucket(const Hit* hits, const unsigned long long* nh_dev, uint64_t nh_cap,
                              uint32_t big, uint32_t* bb, uint32_t* bb_off, void* scan_tmp,
                              size_t scan_bytes, Hit* out, hipStream_t s);
// list-segment verification of the lists with >= big candidates (hits big[0 .. nbig), segp =
// exclusive scan of ceil(count / seg_members), nseg segments, `chunk` segments per wave chunk; first:
// seg_chunks(nseg, chunk) u32 of scratch; ticket: the zeroed word of the first of kTicketLines counter
// lines, or nullptr when the grid has a wave for every chunk)
// list segments of `members` candidates each (seg_members: what k_verify_segs expects)
int seg_members(int y_maxlen, int tau, int lane_cands);
hipError_t launch_seg_counts(const Hit* big, uint64_t nbig, int members, uint32_t* segs,
                             hipStream_t s);
// the same through the parts' automata: tau <= 4, one candidate per lane, strings of up to kAutoMaxLen
constexpr int kAutoMaxLen = 47;
hipError_t launch_verify_auto(const VerifyParams& V, const Hit* big, uint64_t nbig,
                              const uint32_t* segp, uint64_t nseg, const uint32_t* first, uint64_t nchunks,
                              uint32_t chunk, uint64_t waves, unsigned long long* ticket,
                              hipStream_t s);
hipError_t launch_verify_segs(const VerifyParams& V, const Hit* big, const uint32_t* segp,
                              uint64_t nbig, uint64_t nseg, uint32_t* first, int chunk,
                              int lane_cands, int grid, unsigned long long* ticket,
                              hipStream_t s);
uint64_t seg_chunks(uint64_t nseg, int chunk);
// shared-prefix verification (Sec. 5.3) of the big lists: a lane takes a chain of up to
// kChainMembers consecutive members of a content-ordered list.  chains: per big hit, its chain
// count (u32, launch_chain_counts); cprefix: exclusive u64 scan of it (nbig + 1); first:
// (nchains + 63) / 64 u32 of scratch.  Supports tau + 1 <= kShareMaxW (the caller checks).
constexpr int kChainMembers = 16;
constexpr int kShareMaxW = 9;
hipError_t launch_chain_counts(const Hit* big, uint64_t nbig, const uint16_t* x_slen,
                               const uint32_t* runlen, int self, uint32_t* chains, hipStream_t s);
hipError_t launch_verify_chains(const VerifyParams& V, const Hit* big,
                                const unsigned long long* cprefix, uint64_t nbig,
                                uint64_t nchains, uint32_t* first, int grid, hipStream_t s);
// content order of the entries: (key, first 8 bytes of the string, g) -> svals; list lengths at
// each list's first entry -> runlen
hipError_t launch_prefix8_keys(const DevSet& S, const uint32_t* vals, int64_t E, uint64_t* keys,
                               uint32_t* idx, hipStream_t s);
hipError_t launch_gather_keys(const uint64_t* keys, const uint32_t* idx, int64_t E,
                              uint64_t* out, hipStream_t s);
hipError_t launch_gather_vals(const uint32_t* vals, const uint32_t* idx, int64_t E, uint32_t* out,
                              hipStream_t s);
hipError_t launch_run_lengths(const uint32_t* runstart, uint32_t nruns, uint32_t E,
                              uint32_t* runlen, hipStream_t s);
hipError_t launch_verify_batched(const VerifyParams& V, uint32_t* first, int grid, hipStream_t s);
// long-string verification of the small-list hits (V.hits[0 .. V.nhits), ncand candidates,
// uniform tau + 1 <= kLongMaxW, no per-query tau): candidates in slot order, the left parts' first
// rows a candidate a lane, then a diagonal a lane.  grid: blocks.  scratch: long_scratch_bytes(ncand)
// bytes.
constexpr int kLongMinLen = 128;
constexpr int kLongMaxW = 33;
size_t long_scratch_bytes(uint64_t ncand);
hipError_t launch_verify_long(const VerifyParams& V, uint64_t ncand, void* scratch, int grid,
                              hipStream_t s);
// wave chunks of 64 * rounds candidates (rounds in [1, kBatchedRoundsMax])
uint64_t batched_chunks(uint64_t ncand, int rounds);
// A query batch with every size in device memory (a serving slot's captured pipeline, a small
// pj_query, pj_query_noalloc).  counters (zeroed by the upload of the batch tables): [0] hits
// [1] candidates [2] selected [3] accepted [4] cells [5] guard misses [6] side pairs [7] unused;
// bcounts after them: [0] hits [1] candidates [2] wave chunks [3] overflow flags (1 hits, 2
// candidates, 4 accepted, 8 sort) [4] rounds of 64 candidates per chunk.  result: the 8 counters, 4
// bcounts, the number of pairs, then the batch's sorted distinct (query id << 32 | indexed id)
// pairs.
struct GraphBatch {
    ProbeParams probe;          // nx_dev set; hits/hit_cap/counters set
    int probe_grid;
    VerifyParams verify;        // dev_counts = bcounts; prefix/out/out_cap/counters set
    int verify_grid;
    unsigned long long* bcounts;
    uint32_t* first;            // [max(kBatchWaves, cand_cap / 1024) + 1]
    uint64_t cand_cap;          // candidates beyond it overflow
    // short side path (indexed strings shorter than tau_max + 1), y_count == 0: none
    uint32_t y_first, y_count;
    const uint8_t* y_arena; const uint16_t* y_slen; const int32_t* y_lenstart;
    const int64_t* y_gbase;
    // output
    const int32_t* xperm; const int32_t* yperm;
    unsigned long long* result;
};
constexpr int kGraphSortCap = 8192;     // accepted pairs a captured batch can sort
constexpr int kBatchWaves = 8192;       // wave chunks a batch is spread over before they grow
constexpr int kBatchResultHead = 13;    // words of a result before its pairs
// the probe, then the rest of the batch
hipError_t launch_graph_probe(const GraphBatch& G, hipStream_t s);
hipError_t launch_graph_verify(const GraphBatch& G, hipStream_t s);
hipError_t launch_short_path(const DevSet& P, const DevSet& Y, int tau, int self,
                             const int32_t* q_tau, uint64_t* out, uint64_t out_cap,
                             unsigned long long* counters, hipStream_t s);
hipError_t launch_pairs_to_keys(const uint64_t* acc, uint64_t m, const int32_t* xperm,
                                const int32_t* yperm, int self, int bbits, uint64_t* keys,
                                hipStream_t s);
// at most kSmallPairs accepted (gx, gy) -> sorted distinct id pairs a, b and their number, in one
// block
constexpr int kSmallPairs = 4096;
hipError_t launch_small_pairs(const uint64_t* acc, uint64_t m, const int32_t* xperm,
                              const int32_t* yperm, int self, int bbits, int32_t* a, int32_t* b,
                              uint32_t* count, hipStream_t s);

// streamed self-joins: window pairs -> global keys (halo-only pairs as a counted sentinel that
// sorts last); sorted keys -> pair arrays
hipError_t launch_window_keys(const int32_t* a, const int32_t* b, uint64_t m, const int32_t* ids,
                              const int32_t* offs, int min_len, int bbits, uint64_t* keys,
                              unsigned long long* dropped, hipStream_t s);
hipError_t launch_split_keys(const uint64_t* keys, uint64_t m, int bbits, int32_t* a, int32_t* b,
                             hipStream_t s);
// p[0 .. n) = v (a kernel: capturable in a graph, unlike a memset node)
hipError_t launch_fill_words(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s);
// *sum = checksum of the device string set (offsets[0..n], bytes[0..min(offsets[n], cap)))
hipError_t launch_set_checksum(const int32_t* offs, int64_t n, const uint8_t* bytes, int64_t cap,
                               unsigned long long* sum, hipStream_t s);
hipError_t launch_gather_i32(const int32_t* in, const int32_t* perm, int64_t n, int32_t* out,
                             hipStream_t s);

// ---- device-wide primitives (pj_sort.hip) ----
// Exclusive scans; out has n + 1 entries (out[n] = total).
hipError_t scan_u32_to_u32(const uint32_t* in, uint32_t* out, uint64_t n, void* tmp,
                           size_t tmp_bytes, hipStream_t s);
hipError_t scan_u32_to_u64(const uint32_t* in, unsigned long long* out, uint64_t n, void* tmp,
                           size_t tmp_bytes, hipStream_t s);
size_t scan_tmp_bytes(uint64_t n);

// Stable LSD radix sort by the low `bits` bits of the keys, 8 bits per pass.  Buffers ping-pong;
// returns in *result_in_alt whether the sorted data ended in the alternate buffers (it does when
// radix_passes(bits) is odd).
hipError_t radix_sort_u64(uint64_t* keys, uint32_t* vals, uint64_t* keys_alt,
                          uint32_t* vals_alt, uint64_t n, int bits, void* tmp, size_t tmp_bytes,
                          bool* result_in_alt, hipStream_t s);
hipError_t radix_sort_u32(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt,
                          uint32_t* vals_alt, uint64_t n, int bits, void* tmp, size_t tmp_bytes,
                          bool* result_in_alt, hipStream_t s);
int radix_passes(int bits);
size_t radix_tmp_bytes(uint64_t n);

// Heads of runs of equal keys, in order (tmp: scan_tmp_bytes(n)): the first entry of every run;
// the distinct sorted pair keys as id columns.  *count = their number.
hipError_t launch_run_starts(const uint64_t* keys, uint64_t n, void* tmp, size_t tmp_bytes,
                             uint32_t* runstart, uint32_t* count, hipStream_t s);
hipError_t launch_unique_pairs(const uint64_t* keys, uint64_t n, int bbits, void* tmp,
                               size_t tmp_bytes, int32_t* a, int32_t* b, uint32_t* count,
                               hipStream_t s);

}  // namespace pj
