// C ABI of libparrot_attn: argument checks, work sizing and kernel launches.
// Everything here runs on host scalars; no call reads device memory except
// parrot_validate_inputs, which synchronises on purpose.
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <mutex>
#include <string>

#include "parrot_attn.h"
#include "ceiling.h"
#include "common.h"
#include "errors.h"
#include "prefill_args.h"
#include "prefill_shape.h"

namespace {

thread_local std::string g_err;

parrot_status fail(parrot_status s, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

}  // namespace

namespace parrot {

parrot_status set_error(parrot_status s, const char* fmt, ...) {
  if (s == PARROT_OK) {
    g_err.clear();
    return s;
  }
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

}  // namespace parrot

namespace {

long ceil_div(long a, long b) { return (a + b - 1) / b; }

bool aligned(const void* p, size_t n) { return (reinterpret_cast<uintptr_t>(p) % n) == 0; }

// Chunk sizes and slot counts.  Chunks are whole 16-token blocks.  A prefix
// chunk is one prefix-group workgroup's work (see prefix_chunk below).
#ifndef PARROT_PREFIX_CHUNK
#define PARROT_PREFIX_CHUNK 256
#endif
#ifndef PARROT_SPLITKV_WGS_PER_CU
#define PARROT_SPLITKV_WGS_PER_CU 2     // split-KV workgroups (4 waves each) per CU
#endif
#ifndef PARROT_SPLITKV_MIN_BLOCKS
#define PARROT_SPLITKV_MIN_BLOCKS 2
#endif
#ifndef PARROT_SPLITKV_HPW
#define PARROT_SPLITKV_HPW 2            // heads per split-KV wave on the shared path (1 or 2)
#endif
#ifndef PARROT_SPLITKV_WGS_PER_CU_HPW2
#define PARROT_SPLITKV_WGS_PER_CU_HPW2 1
#endif
constexpr int kPrefixChunk = PARROT_PREFIX_CHUNK;
constexpr int kPrefixChunkMax = 1024;   // the prefix role's table stage holds 64 blocks
constexpr int kSplitkvWgsPerCu = PARROT_SPLITKV_WGS_PER_CU;
constexpr int kSplitkvMinBlocks = PARROT_SPLITKV_MIN_BLOCKS;
constexpr int kSplitkvHpw = PARROT_SPLITKV_HPW;
constexpr int kSplitkvWgsPerCuHpw2 = PARROT_SPLITKV_WGS_PER_CU_HPW2;

// Compute units of the current device (cached per device; no device sync).
int num_cus() {
  static std::atomic<int> cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int v = cache[dev].load(std::memory_order_relaxed);
  if (v == 0) {
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
    cache[dev].store(v, std::memory_order_relaxed);
  }
  return v;
}

// Heads per split-KV wave on the shared path.  Two adjacent heads give each
// wave one contiguous 8 KiB piece per tensor and block instead of 4 KiB: a read
// probe over random 128 KiB blocks reaches 7.0 TB/s with 8 KiB pieces at four
// waves per CU against 6.7 TB/s with 4 KiB pieces at eight (the same bytes in
// flight), and the own-token stream ran 2-3.5 % faster on the 32-layer mixed,
// system-prompt and map-reduce workloads.  Its kernel runs two waves per SIMD
// (twice the registers per fetched block), which leaves fewer slots for the
// prefix workgroups once the own-token stream drains, so it is taken when the
// prefix tokens (bound: groups x max_prefix_len) are at most half the own
// tokens (bound: requests x max_suffix_len): at a 16384-token prefix over 32
// requests it was 2.3 % slower.  Even head counts and 16-bit caches only (an
// fp32 block is twice the registers).  Decode with append takes the same
// layout as the plain call, so the two give the same bits.
int splitkv_hpw(const parrot_problem* p, bool shared) {
  if (kSplitkvHpw != 2 || !shared || p->num_heads % 2 != 0 || p->dtype == PARROT_DTYPE_F32) return 1;
  const double prefix_tokens = (double)p->num_groups * p->max_prefix_len;
  const double own_tokens = (double)p->num_requests * p->max_suffix_len;
  return 2.0 * prefix_tokens <= own_tokens ? 2 : 1;
}

// Split-KV workgroups of a decode launch: a fixed number per CU, and at least
// one wave per head group.
long splitkv_workgroups(int heads, int hpw = 1) {
  long n = (long)num_cus() * (hpw == 2 ? kSplitkvWgsPerCuHpw2 : kSplitkvWgsPerCu);
  const long hg = heads / hpw;
  if (n * parrot::kSkvWaves < hg) n = ceil_div(hg, parrot::kSkvWaves);
  return n;
}

// Column groups of the split-KV role (waves per head group).
long splitkv_groups(int heads, int hpw) {
  return splitkv_workgroups(heads, hpw) * parrot::kSkvWaves / (heads / hpw);
}

// Prefix chunk length.  One prefix-group workgroup streams one chunk of one
// head for up to 64 members, about two 16 KiB stages in flight, so its run time
// grows with the chunk; every chunk also costs each member one partial result
// written and merged.  With n(c) = max_prefix_len * groups * heads * query
// tiles / c workgroups for chunk c (an upper bound: the host only knows the
// maximum prefix length), measured on MI355X:
//  * n(1024) <= CUs: the smallest c in {256, 512, 1024} with n(c) <= CUs; all
//    prefix workgroups then run alongside the own-token stream from the start;
//  * CUs < n(1024) <= 2 CUs: c = 512, so that the workgroups that start late
//    (once the own-token stream drains) are short;
//  * otherwise c = 1024 (many rounds anyway; fewest partial results).
// The smallest chunk is 256 tokens, unless the own-token stream is too short to
// cover a 256-token chunk: a chunk costs about one memory round trip (taken as
// 1.5 us) per 32-token stage, and the stream about its bytes at 5 TB/s, so the
// chunk then shrinks to the stages the stream covers (down to one stage: 32
// tokens).  Measured: a 4-request, 128-token fp32 group (own tokens ~100)
// 16.3 -> 10.7 us per call; the benchmark workloads keep their chunks.
// `any_stream`: the chunk for the shortest own-token stream (the smallest the
// rule can give for these prefix sizes), which sizes the workspace so that it
// does not shrink when requests or own tokens are added.
int prefix_chunk(const parrot_problem* p, int qtiles, bool any_stream = false) {
  if (p->num_groups <= 0) return kPrefixChunk;
  const double work = (double)p->max_prefix_len * p->num_groups * p->num_heads * qtiles;
  const double cus = num_cus();
  const double elt = p->dtype == PARROT_DTYPE_F32 ? 4.0 : 2.0;
  const double own_bytes = (double)p->num_requests * p->max_suffix_len * 2.0 * p->num_heads * p->head_dim * elt;
  const double stream_stages = any_stream ? 0.0 : own_bytes / 5e12 / 1.5e-6;
  int cp = kPrefixChunk;
  while (cp > 32 && cp / 32 > stream_stages) cp /= 2;
  if (work / kPrefixChunkMax <= cus) {
    while (cp < kPrefixChunkMax && work / cp > cus) cp *= 2;
  } else if (work / kPrefixChunkMax <= 2 * cus) {
    cp = std::max(cp, kPrefixChunkMax / 2);
  } else {
    cp = std::max(cp, kPrefixChunkMax);
  }
  return cp;
}

parrot_status check_problem(const parrot_problem* p, parrot::Plan* pl) {
  if (!p) return fail(PARROT_ERR_INVALID_ARGUMENT, "problem is NULL");
  if (p->num_requests < 0) return fail(PARROT_ERR_INVALID_ARGUMENT, "num_requests %d < 0", p->num_requests);
  if (p->num_heads < 1) return fail(PARROT_ERR_INVALID_ARGUMENT, "num_heads %d < 1", p->num_heads);
  if (p->num_groups < 0) return fail(PARROT_ERR_INVALID_ARGUMENT, "num_groups %d < 0", p->num_groups);
  if (p->dtype != PARROT_DTYPE_F32 && p->dtype != PARROT_DTYPE_F16 && p->dtype != PARROT_DTYPE_BF16)
    return fail(PARROT_ERR_UNSUPPORTED, "dtype %d is not f32, f16 or bf16", (int)p->dtype);
  if (p->head_dim != 64 && p->head_dim != 128)
    return fail(PARROT_ERR_UNSUPPORTED, "head_dim %d (built for 64 and 128)", p->head_dim);
  if (p->block_size != parrot::kBlock)
    return fail(PARROT_ERR_UNSUPPORTED, "block_size %d (built for 16)", p->block_size);
  if (!std::isfinite(p->sm_scale)) return fail(PARROT_ERR_INVALID_ARGUMENT, "sm_scale is not finite");
  if (p->max_suffix_len < 0) return fail(PARROT_ERR_INVALID_ARGUMENT, "max_suffix_len %d < 0", p->max_suffix_len);
  if (p->max_prefix_len < 0) return fail(PARROT_ERR_INVALID_ARGUMENT, "max_prefix_len %d < 0", p->max_prefix_len);
  const int B = p->block_size;
  if (p->num_groups > 0) {
    if (p->max_prefix_len < 1) return fail(PARROT_ERR_INVALID_ARGUMENT, "max_prefix_len must be >= 1 when num_groups > 0");
    if (p->max_group_size < 1) return fail(PARROT_ERR_INVALID_ARGUMENT, "max_group_size must be >= 1 when num_groups > 0");
    if (p->max_group_size > p->num_requests && p->num_requests > 0)
      return fail(PARROT_ERR_INVALID_ARGUMENT, "max_group_size %d > num_requests %d", p->max_group_size, p->num_requests);
    if (p->prefix_table_stride < ceil_div(p->max_prefix_len, B))
      return fail(PARROT_ERR_INVALID_ARGUMENT, "prefix_table_stride %d < ceil(max_prefix_len / block_size) = %ld",
                  p->prefix_table_stride, ceil_div(p->max_prefix_len, B));
    if (p->num_prefix_blocks < 1) return fail(PARROT_ERR_INVALID_ARGUMENT, "num_prefix_blocks must be >= 1 when num_groups > 0");
  }
  if (p->suffix_table_stride < ceil_div(p->max_suffix_len, B) || p->suffix_table_stride < 0)
    return fail(PARROT_ERR_INVALID_ARGUMENT, "suffix_table_stride %d < ceil(max_suffix_len / block_size) = %ld",
                p->suffix_table_stride, ceil_div(p->max_suffix_len, B));
  if (p->num_suffix_blocks < 1) return fail(PARROT_ERR_INVALID_ARGUMENT, "num_suffix_blocks must be >= 1");
  if (p->num_requests > 0 && p->num_groups == 0 && p->max_suffix_len == 0)
    return fail(PARROT_ERR_INVALID_ARGUMENT, "no request can have a non-empty context (no groups, max_suffix_len 0)");

  if (p->max_prefix_depth < 0) return fail(PARROT_ERR_INVALID_ARGUMENT, "max_prefix_depth %d < 0", p->max_prefix_depth);
  if (p->max_prefix_depth > parrot::kMaxDepth)
    return fail(PARROT_ERR_UNSUPPORTED, "max_prefix_depth %d > %d", p->max_prefix_depth, parrot::kMaxDepth);
  pl->depth = p->num_groups > 0 ? std::max(1, (int)p->max_prefix_depth) : 0;
  const long mg = p->num_groups > 0 ? p->max_group_size : 1;
  pl->prefix_waves = 4;
  pl->prefix_qtiles = (int)ceil_div(mg, 16 * pl->prefix_waves);
  pl->cp = prefix_chunk(p, pl->prefix_qtiles);
  pl->skv_min_q = kSplitkvMinBlocks;
  // slots: shared path = prefix chunks + split-KV pieces of the own tokens;
  // per-request path = split-KV pieces of prefix + own tokens.  One stride
  // serves both.  A sequence of n block columns touches at most
  // ceil(n / min_q) + 1 runs of the flat column list, and never more than the
  // G column groups the role has (its piece index is its group minus the
  // group of its first column).
  const long nbp_max = p->num_groups > 0 ? ceil_div(p->max_prefix_len, B) : 0;
  const long nbs_max = ceil_div(p->max_suffix_len, B);
  // the shared path streams one or two heads per wave, the per-request path
  // one; a bound on the pieces covers either
  const long groups = splitkv_groups(p->num_heads, 1);
  const long groups_shared = std::max(groups, splitkv_groups(p->num_heads, splitkv_hpw(p, true)));
  const long pieces_shared = nbs_max > 0 ? std::min(ceil_div(nbs_max, pl->skv_min_q) + 1, groups_shared) : 0;
  const long pieces_naive = std::min(ceil_div(nbp_max + nbs_max, pl->skv_min_q) + 1, groups);
  pl->seg_p = p->num_groups > 0 ? (int)ceil_div(p->max_prefix_len, pl->cp) : 0;
  if (pl->seg_p > 0xFFFF)
    return fail(PARROT_ERR_UNSUPPORTED, "max_prefix_len %d needs %d prefix chunks (at most 65535)",
                p->max_prefix_len, pl->seg_p);
  pl->seg_pre = pl->depth * pl->seg_p;
  pl->seg_s = (int)pieces_shared;
  const long seg = std::max<long>(pl->seg_pre + pieces_shared, pieces_naive);
  pl->seg = (int)seg;
  pl->skv_waves = 0;   // set at launch from the device's CU count
  // the workspace holds the slots of the smallest prefix chunk any own-token
  // stream could select (at least this call's): its size never drops when
  // num_requests or max_suffix_len grow
  const long seg_p_ws = p->num_groups > 0 ? ceil_div(p->max_prefix_len, prefix_chunk(p, pl->prefix_qtiles, true)) : 0;
  const long seg_ws = std::max<long>(std::max<long>(pl->depth * seg_p_ws + pieces_shared, pieces_naive), seg);

  const double slots = (double)p->num_requests * p->num_heads * seg_ws;
  const double flat = (double)p->num_requests * (double)(nbp_max + nbs_max);
  const double grid_b = (double)p->num_groups * pl->seg_p * p->num_heads * pl->prefix_qtiles;
  if (flat > 2e9 || grid_b > 2e9 || slots * p->head_dim * 4.0 > 9e18)
    return fail(PARROT_ERR_UNSUPPORTED, "problem too large for one launch (%.3g blocks)", flat);
  const size_t n_slots = (size_t)p->num_requests * p->num_heads * seg_ws;
  auto align256 = [](size_t x) { return (x + 255) & ~(size_t)255; };
  pl->o_bytes = align256(n_slots * p->head_dim * sizeof(float));
  pl->lse_bytes = align256(n_slots * sizeof(float));
  pl->info_bytes = align256((size_t)p->num_requests * parrot::kMetaInts * sizeof(int32_t));
  pl->total_bytes = p->num_requests > 0 ? pl->o_bytes + pl->lse_bytes + pl->info_bytes : 0;
  return PARROT_OK;
}

// The workspace layout of one shared-path call sized for that call alone: the
// prefix chunks of this call's chunk size and its split-KV pieces, with no
// slots reserved for the per-request path or for smaller chunks (used where
// the workspace is the library's own fixed array and is laid out afresh on
// every call).
void exact_shared_layout(const parrot_problem* p, parrot::Plan* pl) {
  pl->seg = pl->seg_pre + pl->seg_s;
  const size_t n_slots = (size_t)p->num_requests * p->num_heads * pl->seg;
  auto align256 = [](size_t x) { return (x + 255) & ~(size_t)255; };
  pl->o_bytes = align256(n_slots * p->head_dim * sizeof(float));
  pl->lse_bytes = align256(n_slots * sizeof(float));
  pl->info_bytes = align256((size_t)p->num_requests * parrot::kMetaInts * sizeof(int32_t));
  pl->total_bytes = p->num_requests > 0 ? pl->o_bytes + pl->lse_bytes + pl->info_bytes : 0;
}

hipEvent_t ev(void* p) { return reinterpret_cast<hipEvent_t>(p); }

parrot_status hip_ok(hipError_t e, const char* what) {
  if (e != hipSuccess) return fail(PARROT_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
  return PARROT_OK;
}

parrot_status launched(hipError_t e, const char* what) {
  if (e != hipSuccess) return fail(PARROT_ERR_HIP, "%s launch failed: %s", what, hipGetErrorString(e));
  return PARROT_OK;
}

// End of a call whose single kernel wrote the output: the merge's trace events,
// if asked for, bracket nothing.
parrot_status no_merge(const parrot_trace& tr, hipStream_t s) {
  parrot_status st = PARROT_OK;
  if (tr.merge_start) st = hip_ok(hipEventRecord(ev(tr.merge_start), s), "hipEventRecord");
  if (st == PARROT_OK && tr.merge_stop) st = hip_ok(hipEventRecord(ev(tr.merge_stop), s), "hipEventRecord");
  if (st == PARROT_OK) g_err.clear();
  return st;
}

#define PARROT_TRY(x) do { parrot_status _s = (x); if (_s != PARROT_OK) return _s; } while (0)

// `g_decode_path` (per thread, set through parrot_test_decode_path) overrides the
// estimate below for tests and tuning: 0 two kernels; 1, 4 or 8 one launch (with
// the rule's, four or eight waves per workgroup) wherever its lists fit.
thread_local int g_decode_path = -1;

// Waves per workgroup of the one-launch decode path (direct.hip), or 0 where the
// partial-result and merge kernels are expected to be faster.  Every side is
// estimated in microseconds from the bounds in `p`, so every entry point of a
// path makes the same choice for the same problem.  The figures are fits to 620
// calls on MI355X (1-128 requests over none, one, some or a group each, even and
// ragged lengths of 1-4096 tokens, 4-40 heads, every dtype and head size, shared,
// appending, nested and per request), each timed with its KV still in the 256 MB
// cache and without:
//  * bytes: a call reads the own tokens and each distinct prefix (at most one per
//    request and level) from memory, whatever path it takes, and a prefix's other
//    readers take it from the caches at 19-22 TB/s.  Lengths are bounds: the mean
//    own length is taken as 0.46 of it, that of several prefixes as 0.64.
//  * one launch: its longest context at 52 KB/us for a workgroup of eight waves
//    (37 for four; rows under 512 bytes count as 512), or the bytes at 3.4 TB/s
//    (3.3), whichever is longer: nothing balances ragged contexts.  4.2 us (3.9)
//    without any, 2.3 us (1.2) more per further workgroup of a CU.
//  * two kernels: 10 us, the bytes at 6.9 TB/s (fp32 prefixes 1.3, with 64-wide
//    heads 4) or the first prefix chunk's chain (0.11 us a token in fp32, 0.064
//    64-wide, 0.016 in 16 bits), and 0.17 us per piece of the longest own tokens
//    that the merge reads.
// Eight waves also above one workgroup per CU where their estimate is lower (257
// to 512 workgroups of long contexts); four never below, where they are slower or
// within 5 %.
// Of the 620 calls one is more than 3 % slower than on two kernels with its KV in
// the cache and 31 (at most 17 %) with it in memory; on the whole 1.30x and 1.19x.
// Measured, two kernels / one, 32 heads of 128, 16 bits: 8 requests of 300 tokens
// 15.3 / 10.8 us, 8 of 1000 28.6 / 29.6, 32 of 300 33.1 / 40.0, 8 on one 500-token
// prefix 10.9 / 9.3, on a 2000-token one 14.9 / 19.6, on four of 1000 18.7 / 16.0 (20.7
// / 22.2 from memory), 4 on three of 3000 35.7 / 46.1; 29 on 22 of 1062, 40 heads,
// 131 / 177; 39 on 20 of 2000, 8 heads, 47 / 62.
int direct_waves(const parrot_problem* p, const parrot::Plan& pl, bool shared) {
  const int depth = p->num_groups > 0 ? std::max(1, (int)p->max_prefix_depth) : 0;
  const double pre = p->num_groups > 0 ? p->max_prefix_len : 0.0, own = p->max_suffix_len;
  const double R = p->num_requests, H = p->num_heads, cus = num_cus();
  const double wgs = R * H;
  if (pre > parrot::kDirectMaxTokens || own > parrot::kDirectMaxTokens || wgs > parrot::kDirectMaxWgs ||
      g_decode_path == 0)
    return 0;
  if (g_decode_path > 1) return g_decode_path;
  if (g_decode_path == 1) return wgs <= cus ? 8 : 4;

  const bool f32 = p->dtype == PARROT_DTYPE_F32, wide = p->head_dim == 128;
  const double row = 2.0 * p->head_dim * (f32 ? 4.0 : 2.0);   // K and V of one token and head
  const double distinct = std::min((double)p->num_groups, R * depth);
  const double own_tokens = R * own * (R > 1 ? 0.46 : 1.0);
  const double pre_mean = pre * (distinct > 1 ? 0.64 : 1.0);
  const double own_bytes = own_tokens * H * row, pre_bytes = distinct * pre_mean * H * row;
  const double repeats = std::max(0.0, R * depth - distinct) * pre_mean * H * row;

  const double longest = (depth * pre + own) * std::max(row, 512.0), more = std::max(0.0, wgs / cus - 1.0);
  const double one8 = 4.2 + std::max(longest / 52e3, (own_bytes + pre_bytes) / 3.4e6 + repeats / 22e6) + 2.3 * more;
  const double one4 = 3.9 + std::max(longest / 37e3, (own_bytes + pre_bytes) / 3.3e6 + repeats / 22e6) + 1.2 * more;

  // column groups and columns of the split-KV role, and so pieces per sequence
  const int hpw = splitkv_hpw(p, shared);
  const double cols = (own_tokens + (shared ? 0.0 : R * depth * pre_mean)) / parrot::kBlock;
  const double run = std::max((double)pl.skv_min_q, cols / splitkv_groups(p->num_heads, hpw));
  const double pieces = (own + (shared ? 0.0 : pre)) / parrot::kBlock / run;
  double two = 10.0 + 0.17 * pieces;
  if (shared) {
    const double chain = p->num_groups > 0 ? std::min(pre, (double)pl.cp) * (!f32 ? 0.016 : wide ? 0.11 : 0.064) : 0.0;
    two += std::max(own_bytes / 6.9e6 + pre_bytes / (!f32 ? 6.9e6 : wide ? 1.3e6 : 4.0e6), chain);
  } else {
    two += (own_bytes + pre_bytes) / 6.9e6 + repeats / 19e6;
  }
  const int waves = wgs <= cus || one8 <= one4 ? 8 : 4;
  return (waves == 8 ? one8 : one4) < two ? waves : 0;
}

// shared: prefix-group role for the prefixes (else the split-KV role reads
// them per request); parents: nested groups (shared path only; NULL = flat).
// k_new / v_new (both or neither): append this step's token to the suffix
// pools (which are then written) while attending.
parrot_status decode(bool shared, const parrot_problem* p, const void* q, const void* prefix_k,
                     const void* prefix_v, const void* suffix_k, const void* suffix_v,
                     const int32_t* ptab, const int32_t* plen, const int32_t* parents,
                     const int32_t* stab, const int32_t* slen, const int32_t* gid, void* out,
                     float* lse, void* workspace, size_t workspace_bytes, void* stream,
                     const parrot_trace* trace, const void* k_new = nullptr,
                     const void* v_new = nullptr, bool exact = false) {
  parrot::Plan pl;
  PARROT_TRY(check_problem(p, &pl));
  if (exact) exact_shared_layout(p, &pl);
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const parrot_trace none = {nullptr, nullptr, nullptr, nullptr};
  const parrot_trace& tr = trace ? *trace : none;
  if (p->num_requests == 0) {
    g_err.clear();
    return PARROT_OK;
  }
  struct { const void* ptr; const char* name; size_t align; } req[] = {
      {q, "q", 16}, {suffix_k, "suffix_k", 16}, {suffix_v, "suffix_v", 16},
      {stab, "suffix_block_tables", 4}, {slen, "suffix_lens", 4}, {gid, "group_ids", 4},
      {out, "out", 16}, {lse, "lse", 4}, {workspace, "workspace", 256}};
  for (auto& r : req) {
    if (!r.ptr) return fail(PARROT_ERR_INVALID_ARGUMENT, "%s is NULL", r.name);
    if (!aligned(r.ptr, r.align)) return fail(PARROT_ERR_INVALID_ARGUMENT, "%s is not %zu-byte aligned", r.name, r.align);
  }
  if (p->num_groups > 0) {
    struct { const void* ptr; const char* name; size_t align; } preq[] = {
        {prefix_k, "prefix_k", 16}, {prefix_v, "prefix_v", 16},
        {ptab, "prefix_block_tables", 4}, {plen, "prefix_lens", 4}};
    for (auto& r : preq) {
      if (!r.ptr) return fail(PARROT_ERR_INVALID_ARGUMENT, "%s is NULL", r.name);
      if (!aligned(r.ptr, r.align)) return fail(PARROT_ERR_INVALID_ARGUMENT, "%s is not %zu-byte aligned", r.name, r.align);
    }
  }
  if (k_new || v_new) {
    struct { const void* ptr; const char* name; } areq[] = {{k_new, "k_new"}, {v_new, "v_new"}};
    for (auto& r : areq) {
      if (!r.ptr) return fail(PARROT_ERR_INVALID_ARGUMENT, "%s is NULL", r.name);
      if (!aligned(r.ptr, 16)) return fail(PARROT_ERR_INVALID_ARGUMENT, "%s is not 16-byte aligned", r.name);
    }
  }
  if (workspace_bytes < pl.total_bytes)
    return fail(PARROT_ERR_WORKSPACE_TOO_SMALL, "workspace is %zu bytes, need %zu", workspace_bytes, pl.total_bytes);

  float* o_part = reinterpret_cast<float*>(workspace);
  float* lse_part = reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) + pl.o_bytes);
  int* merge_meta = reinterpret_cast<int*>(reinterpret_cast<char*>(workspace) + pl.o_bytes + pl.lse_bytes);
  const float scale_log2 = p->sm_scale * parrot::kLog2e;
  const int D = p->head_dim, dt = (int)p->dtype;

  if (const int waves = direct_waves(p, pl, shared)) {
    parrot::DirectArgs a{};
    a.q = q; a.pk = prefix_k; a.pv = prefix_v; a.sk = suffix_k; a.sv = suffix_v;
    a.ptab = ptab; a.plen = plen; a.stab = stab; a.slen = slen; a.gid = gid;
    a.parents = parents;
    a.depth = parents ? pl.depth : 1;
    a.k_new = k_new; a.v_new = v_new;
    a.app_k = const_cast<void*>(suffix_k); a.app_v = const_cast<void*>(suffix_v);
    a.out = out; a.lse = lse;
    a.R = p->num_requests; a.H = p->num_heads; a.NG = p->num_groups;
    a.pstride = p->prefix_table_stride; a.sstride = p->suffix_table_stride;
    a.max_p = p->max_prefix_len; a.max_s = p->max_suffix_len;
    a.npblk = p->num_groups > 0 ? p->num_prefix_blocks : 1; a.nsblk = p->num_suffix_blocks;
    a.scale_log2 = scale_log2;
    PARROT_TRY(launched(parrot::launch_direct(a, waves, dt, D, s, ev(tr.partials_start), ev(tr.partials_stop)),
                        "decode kernel"));
    return no_merge(tr, s);
  }

  const bool run_prefix = shared && p->num_groups > 0 && pl.seg_p > 0;
  {
    parrot::PartialsArgs pa{};
    parrot::SplitKVArgs& a = pa.skv;
    a.q = q; a.pk = prefix_k; a.pv = prefix_v; a.sk = suffix_k; a.sv = suffix_v;
    a.ptab = ptab; a.plen = plen; a.stab = stab; a.slen = slen; a.gid = gid;
    a.parents = shared ? parents : nullptr;
    a.depth = parents ? pl.depth : 1;
    a.k_new = k_new; a.v_new = v_new;
    a.app_k = const_cast<void*>(suffix_k); a.app_v = const_cast<void*>(suffix_v);
    a.o_part = o_part; a.lse_part = lse_part; a.merge_meta = merge_meta;
    a.R = p->num_requests; a.H = p->num_heads; a.NG = p->num_groups;
    a.pstride = p->prefix_table_stride; a.sstride = p->suffix_table_stride;
    a.max_p = p->max_prefix_len; a.max_s = p->max_suffix_len;
    a.npblk = p->num_groups > 0 ? p->num_prefix_blocks : 1; a.nsblk = p->num_suffix_blocks;
    a.seg = pl.seg; a.seg_pre = shared ? pl.seg_pre : 0; a.cp = pl.cp;
    a.with_prefix = shared ? 0 : 1;
    // a fixed grid of split-KV workgroups per CU, at least one wave per head group
    a.hpw = splitkv_hpw(p, shared);
    pa.n_skv = (int)splitkv_workgroups(a.H, a.hpw);
    a.nwaves = pa.n_skv * parrot::kSkvWaves;
    a.min_q = pl.skv_min_q;
    a.scale_log2 = scale_log2;
    if (run_prefix) {
      parrot::PrefixArgs& b = pa.pre;
      b.q = q; b.pk = prefix_k; b.pv = prefix_v; b.ptab = ptab; b.plen = plen; b.gid = gid;
      b.parents = parents;
      b.depth = parents ? pl.depth : 1;
      b.o_part = o_part; b.lse_part = lse_part;
      b.R = p->num_requests; b.H = p->num_heads; b.NG = p->num_groups;
      b.pstride = p->prefix_table_stride; b.max_p = p->max_prefix_len; b.npblk = p->num_prefix_blocks;
      b.seg = pl.seg; b.seg_p = pl.seg_p; b.cp = pl.cp; b.qtiles = pl.prefix_qtiles;
      b.scale_log2 = scale_log2;
      pa.n_pre = p->num_groups * pl.seg_p * p->num_heads * pl.prefix_qtiles;
    }
    // The split-KV role holds its per-request scan in LDS for up to 4096
    // requests (1024 on the per-request path), so a larger batch is streamed in
    // slices of that many requests, one launch each (every per-request pointer
    // moved to the slice); the prefix-group role covers every request in the
    // first launch, and one merge follows.  The trace brackets all of them.
    const int R = p->num_requests, H = p->num_heads;
    const size_t elt = p->dtype == PARROT_DTYPE_F32 ? 4 : 2;
    const int most = shared ? parrot::kMaxRequests : parrot::kMaxRequestsPrefix;
    for (int r0 = 0; r0 < R; r0 += most) {
      const int rn = std::min(most, R - r0);
      parrot::PartialsArgs slice = pa;
      parrot::SplitKVArgs& c = slice.skv;
      const size_t rows = (size_t)r0 * H;
      c.q = static_cast<const char*>(q) + rows * D * elt;
      c.stab = stab + (size_t)r0 * p->suffix_table_stride;
      c.slen = slen + r0;
      c.gid = gid + r0;
      if (k_new) {
        c.k_new = static_cast<const char*>(k_new) + rows * D * elt;
        c.v_new = static_cast<const char*>(v_new) + rows * D * elt;
      }
      c.o_part = o_part + rows * pl.seg * D;
      c.lse_part = lse_part + rows * pl.seg;
      c.merge_meta = merge_meta + (size_t)r0 * parrot::kMetaInts;
      c.R = rn;
      if (r0 > 0) slice.n_pre = 0;
      const bool first = r0 == 0, last = r0 + rn == R;
      PARROT_TRY(launched(parrot::launch_partials(slice, dt, D, s,
                                                  first ? ev(tr.partials_start) : nullptr,
                                                  last ? ev(tr.partials_stop) : nullptr),
                          "partials kernel"));
    }
  }
  {
    parrot::MergeArgs a{};
    a.o_part = o_part; a.lse_part = lse_part; a.merge_meta = merge_meta;
    a.out = out; a.lse = lse;
    a.R = p->num_requests; a.H = p->num_heads;
    a.seg = pl.seg; a.seg_p = pl.seg_p; a.seg_pre = shared ? pl.seg_pre : 0;
    PARROT_TRY(launched(parrot::launch_merge(a, dt, D, s, ev(tr.merge_start), ev(tr.merge_stop)),
                        "merge kernel"));
  }
  g_err.clear();
  return PARROT_OK;
}

}  // namespace

extern "C" {

size_t parrot_workspace_bytes(const parrot_problem* p) {
  parrot::Plan pl;
  if (check_problem(p, &pl) != PARROT_OK) return (size_t)-1;
  g_err.clear();
  return pl.total_bytes;
}

parrot_status parrot_shared_prefix_decode(
    const parrot_problem* p, const void* q, const void* prefix_k, const void* prefix_v,
    const void* suffix_k, const void* suffix_v, const int32_t* prefix_block_tables,
    const int32_t* prefix_lens, const int32_t* suffix_block_tables, const int32_t* suffix_lens,
    const int32_t* group_ids, void* out, float* lse, void* workspace, size_t workspace_bytes,
    void* stream, const parrot_trace* trace) {
  return decode(true, p, q, prefix_k, prefix_v, suffix_k, suffix_v, prefix_block_tables,
                prefix_lens, nullptr, suffix_block_tables, suffix_lens, group_ids, out, lse,
                workspace, workspace_bytes, stream, trace);
}

parrot_status parrot_per_request_decode(
    const parrot_problem* p, const void* q, const void* prefix_k, const void* prefix_v,
    const void* suffix_k, const void* suffix_v, const int32_t* prefix_block_tables,
    const int32_t* prefix_lens, const int32_t* suffix_block_tables, const int32_t* suffix_lens,
    const int32_t* group_ids, void* out, float* lse, void* workspace, size_t workspace_bytes,
    void* stream, const parrot_trace* trace) {
  return decode(false, p, q, prefix_k, prefix_v, suffix_k, suffix_v, prefix_block_tables,
                prefix_lens, nullptr, suffix_block_tables, suffix_lens, group_ids, out, lse,
                workspace, workspace_bytes, stream, trace);
}

parrot_status parrot_shared_prefix_decode_append(
    const parrot_problem* p, const void* q, const void* k_new, const void* v_new,
    const void* prefix_k, const void* prefix_v, void* suffix_k, void* suffix_v,
    const int32_t* prefix_block_tables, const int32_t* prefix_lens,
    const int32_t* suffix_block_tables, const int32_t* suffix_lens, const int32_t* group_ids,
    void* out, float* lse, void* workspace, size_t workspace_bytes, void* stream,
    const parrot_trace* trace) {
  if (p && p->num_requests > 0 && (!k_new || !v_new))
    return fail(PARROT_ERR_INVALID_ARGUMENT, "%s is NULL", k_new ? "v_new" : "k_new");
  return decode(true, p, q, prefix_k, prefix_v, suffix_k, suffix_v, prefix_block_tables,
                prefix_lens, nullptr, suffix_block_tables, suffix_lens, group_ids, out, lse,
                workspace, workspace_bytes, stream, trace, k_new, v_new);
}

parrot_status parrot_nested_prefix_decode(
    const parrot_problem* p, const void* q, const void* prefix_k, const void* prefix_v,
    const void* suffix_k, const void* suffix_v, const int32_t* prefix_block_tables,
    const int32_t* prefix_lens, const int32_t* prefix_parents, const int32_t* suffix_block_tables,
    const int32_t* suffix_lens, const int32_t* group_ids, void* out, float* lse, void* workspace,
    size_t workspace_bytes, void* stream, const parrot_trace* trace) {
  if (p && p->num_requests > 0 && p->num_groups > 0) {
    if (!prefix_parents) return fail(PARROT_ERR_INVALID_ARGUMENT, "prefix_parents is NULL");
    if (!aligned(prefix_parents, 4)) return fail(PARROT_ERR_INVALID_ARGUMENT, "prefix_parents is not 4-byte aligned");
  }
  return decode(true, p, q, prefix_k, prefix_v, suffix_k, suffix_v, prefix_block_tables,
                prefix_lens, p && p->num_groups > 0 ? prefix_parents : nullptr,
                suffix_block_tables, suffix_lens, group_ids, out, lse, workspace,
                workspace_bytes, stream, trace);
}

}  // extern "C"

// ------------------------------------------------------------- test hooks
// Exported for tests and tuning, not declared in parrot_attn.h: the decode path
// of this thread's calls (see g_decode_path; -1 gives the choice back to the
// estimate), and the path a decode or prefill call with these arguments takes.
extern "C" {

void parrot_test_decode_path(int path) {
  g_decode_path = path == 0 || path == 1 || path == 4 || path == 8 ? path : -1;
}

// Waves per workgroup of the one-launch kernel, 0 for two kernels, -1 for
// invalid arguments.
int parrot_test_decode_waves(const parrot_problem* p, int per_request) {
  parrot::Plan pl;
  if (check_problem(p, &pl) != PARROT_OK) return -1;
  return p->num_requests == 0 ? 0 : direct_waves(p, pl, per_request == 0);
}

}  // extern "C"

// ------------------------------------------------------ allocation-free decode
// The partial-result workspace of parrot_shared_prefix_decode_noalloc: one
// fixed array per device, held from the library's load on that device until
// the process ends.  Every call lays its partial results out afresh and
// writes each slot before the merge reads it, so nothing in it has to start
// at zero; calls that overlap on one device share it and race.
static __device__ __align__(256) char scratch[PARROT_STATIC_SCRATCH_BYTES];

namespace {

// Device address of `scratch` on the current device, looked up once per
// device with that device current.  The array's name in host code is only a
// host-side handle; kernels get this address.
parrot_status static_scratch(void** out) {
  static std::atomic<void*> addr[64];
  static std::mutex mu;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(PARROT_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= 64) return fail(PARROT_ERR_UNSUPPORTED, "device %d (at most 64 devices)", dev);
  void* ptr = addr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    std::lock_guard<std::mutex> lock(mu);
    ptr = addr[dev].load(std::memory_order_relaxed);
    if (!ptr) {
      e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !ptr)
        return fail(PARROT_ERR_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
      addr[dev].store(ptr, std::memory_order_release);
    }
  }
  *out = ptr;
  return PARROT_OK;
}

}  // namespace

extern "C" {

parrot_status parrot_shared_prefix_decode_noalloc(
    const parrot_problem* p, const void* q, const void* prefix_k, const void* prefix_v,
    const void* suffix_k, const void* suffix_v, const int32_t* prefix_block_tables,
    const int32_t* prefix_lens, const int32_t* suffix_block_tables, const int32_t* suffix_lens,
    const int32_t* group_ids, void* out, float* lse, void* stream, const parrot_trace* trace) {
  parrot::Plan pl;
  PARROT_TRY(check_problem(p, &pl));
  if (p->num_requests == 0) {
    g_err.clear();
    return PARROT_OK;
  }
  exact_shared_layout(p, &pl);
  if (pl.total_bytes > (size_t)PARROT_STATIC_SCRATCH_BYTES)
    return fail(PARROT_ERR_WORKSPACE_TOO_SMALL,
                "this call needs %zu bytes of partial results; the library's fixed array holds %zu "
                "(use parrot_shared_prefix_decode with a workspace)",
                pl.total_bytes, (size_t)PARROT_STATIC_SCRATCH_BYTES);
  void* ws = nullptr;
  PARROT_TRY(static_scratch(&ws));
  return decode(true, p, q, prefix_k, prefix_v, suffix_k, suffix_v, prefix_block_tables,
                prefix_lens, nullptr, suffix_block_tables, suffix_lens, group_ids, out, lse, ws,
                (size_t)PARROT_STATIC_SCRATCH_BYTES, stream, trace, nullptr, nullptr, true);
}

}  // extern "C"

namespace {

// ------------------------------------------------------------------ prefill
constexpr int kPrefillChunkMax = 8192;   // the prefill tile's table holds 512 blocks
constexpr int kPrefillChunkMin = 256;

struct PrefillPlan {
  int depth, cp, co, seg_p, seg_pre, seg_s, seg, qtiles_p, qtiles_o;
  long n_pre, n_own;
  int waves;     // kPrefillRows: waves per workgroup
  int kind;      // PrefillPlanKind; the single-pass kinds have no partial results and no merge
  size_t o_bytes, lse_bytes, info_bytes, total_bytes;
};

// PARROT_PREFILL_SINGLE_PASS=0 turns the single-pass plans off; =1 takes the
// stacked one and =2 the per-request one wherever the groups are flat, the
// caches 16-bit and the ranges fit the tile's block table (8192 tokens), =3 the
// one without tiles wherever no range exceeds 4096 and one launch holds its
// workgroups, for tests and tuning.  Any other value (or none) leaves the choice
// to the cost estimate below.
int single_pass_setting() {
  const char* e = std::getenv("PARROT_PREFILL_SINGLE_PASS");
  if (e && e[0] >= '0' && e[0] <= '3' && e[1] == 0) return e[0] - '0';
  return -1;
}

// Chunk of a key range of at most `len` tokens: the whole range up to 8192
// tokens (fewest partial results), halved while the items of that chunk size
// (`items_per_chunk` per chunk) would not fill every CU with the three
// workgroups it holds.
int prefill_chunk(long len, double items_per_chunk) {
  int c = kPrefillChunkMax;
  while (c > kPrefillChunkMin && c / 2 >= len) c /= 2;
  const double cus = num_cus();
  while (c > kPrefillChunkMin && items_per_chunk * (double)ceil_div(len, c) < 3 * cus) c /= 2;
  return c;
}

// Estimated microseconds of the three plans for a 16-bit call on flat groups,
// from the bounds the host knows.  The figures are fits to sweeps on MI355X
// (1-64 requests of 1-4000 rows, prefixes of 100-6000 tokens, 8 and 32 heads):
//  * a workgroup alone on its CU takes 0.8 us per 16 KiB stage of keys, and up
//    to three on a CU finish a stage every 0.28 + 0.05 w us together, w the
//    waves with rows (0.33 with one, 0.48 with four);
//  * a tile's set-up and output cost 1 + 0.9 w us of its CU (6 us of latency),
//    each run of rows after a stacked tile's first 1 us (2.5 us of latency);
//  * a launch takes 5 us, the merge of the split plan 4 us more and its partial
//    results (written, then read) pass at 4.5 TB/s (10 within the 256 MB cache).
// Measured, split / stacked / per request: 16 requests of 16-64 rows on a
// 100-token prefix 24 / 26 / 15 us; 64 of 16-64 on 600 tokens 104 / 59 / 84; 64
// of 1-8 on 2000 tokens 51 / 113 / 173; one prompt of 2000 tokens 75 / 59 / 60;
// one of 300 tokens 18 / 12 / 13; 64 of 100-300 on 600 408 / 239 / 229.
struct PrefillCosts { double split, stacked, direct; };

PrefillCosts prefill_costs(const parrot_problem* p, const parrot_prefill_rows* rows,
                           const PrefillPlan& pl) {
  const double H = p->num_heads, R = p->num_requests, T = rows->num_query_rows, cus = num_cus();
  const double st = 4096.0 / p->head_dim;                  // tokens per stage
  const double tile = parrot::kWideRows;
  const double mean_q = T / R;
  const double waves = std::min(4.0, std::ceil(mean_q / 32.0));
  const double per_stage = 0.28 + 0.05 * waves, setup = 1.0 + 0.9 * waves;
  const double full_stage = 0.48, full_setup = 4.6;        // tiles of stacked rows
  // own tokens a tile sees on average: half a whole prompt (plus the tile's
  // own diagonal), or a share of the longest continued one
  const bool whole = rows->max_query_rows >= p->max_suffix_len;
  const double own = std::min<double>(p->max_suffix_len,
                                      !whole ? 0.6 * p->max_suffix_len
                                             : mean_q > tile ? (mean_q + tile) / 2 : mean_q);
  const double own_stages = std::ceil(own / st), max_own = std::ceil(p->max_suffix_len / st);
  const double pre_stages = p->num_groups > 0 ? std::ceil(p->max_prefix_len / st) : 0.0;
  const double tiles_o = R * std::max(1.0, mean_q / tile + (mean_q > tile ? 0.5 : 0.0));
  // (groups that nobody reads make no tiles)
  const double groups = std::min((double)p->num_groups, R * std::max(1, pl.depth));
  const double tiles_p = pl.qtiles_p > 0 ? std::max(T / tile + 0.5 * groups, (double)pl.qtiles_p) : 0.0;
  // the longest tile alone and the load per CU hide most of each other
  auto both = [](double latency, double load) {
    return std::max(6.0 + latency, load) + 0.2 * std::min(6.0 + latency, load);
  };
  PrefillCosts c;
  c.direct = 5.0 + both(0.8 * (pre_stages + max_own),
                        H * tiles_o / cus * ((pre_stages + own_stages) * per_stage + setup));
  if (tiles_p > 0) {
    const double runs = 1.0 + std::min(tile, (double)rows->max_group_rows) / mean_q;
    c.stacked = 5.0 + both(0.8 * pre_stages + runs * (0.8 * own_stages + 2.5),
                           H * tiles_p / cus * ((pre_stages + runs * own_stages) * full_stage +
                                                full_setup + runs));
  } else {
    c.stacked = c.direct;
  }
  const double slots = pl.seg_p + std::max(1.0, pl.seg_s * own / std::max(1, p->max_suffix_len));
  const double partial_bytes = 2.0 * T * H * slots * p->head_dim * 4.0;
  // (its own items run head after head: the last head's long ones end alone)
  const double item_own = std::min(max_own, pl.co / st);
  c.split = 9.0 + partial_bytes / (partial_bytes < 2.5e8 ? 10e6 : 4.5e6) + 0.12 * item_own +
            both(0.8 * std::max(std::min(pre_stages, pl.cp / st), item_own),
                 H * tiles_p / cus * (pre_stages * full_stage + pl.seg_p * full_setup) +
                     H * tiles_o / cus * (own_stages * per_stage + setup));
  return c;
}

// Estimated microseconds of a prefill without tiles (direct.hip: one workgroup
// per row and head that reads the row's whole context), or -1 where it is not
// built.  As for the one-launch decode: 5 us, the longest context at 74 KB/us for
// a workgroup of eight waves (42 for four), or the bytes, whichever is longer:
// each distinct prefix and the own tokens of the requests that bring rows once
// from memory at 5.6 TB/s, every further row's reads from the caches at 28 TB/s
// (12.5 where a head's workgroups spread over more than two XCDs); 1.45 us per
// further workgroup of a CU.  Lengths are bounds: the mean own length is taken as
// 0.55 of it, that of several prefixes as 0.84.  Fitted to 240 calls of 1-64
// requests of 1-300 rows, on none to a prefix each, timed with their KV in the
// cache and without; the tiles' estimates run high where everything waits on
// round trips (13.6 us measured for 21 estimated) and low for the fp32 tile (18
// and 33 us for 14 and 21), hence the factors at the call.
// Measured, tiles / rows: 4 fp32 requests of 16-32 rows on a 128-token prefix, 4
// heads 18.5 / 6.3 us; one fp16 request of 8-16 rows on 600 tokens, 4 heads 14.3 /
// 8.1; 16 of 1-4 rows on 100 tokens, 4 heads 9.3 / 5.4, 32 heads 10.4 / 11.3; 4 of
// 8-16 rows on 100, 32 heads 9.5 / 11.7; two of 5 rows on a prefix of 1405 each, 32
// 64-wide heads 15.9 / 19.6 (17.1 / 28.6 from memory); 5 of 14 rows, own 1054, 4
// heads 13.8 / 18.0 (14.7 / 22.0).
double direct_rows_cost(const parrot_problem* p, long T, int depth) {
  const double pre = p->num_groups > 0 ? p->max_prefix_len : 0.0, own = p->max_suffix_len;
  const double wgs = (double)T * p->num_heads, cus = num_cus();
  if (pre > parrot::kDirectMaxTokens || own > parrot::kDirectMaxTokens || wgs > parrot::kDirectMaxWgs) return -1.0;
  const double row = 2.0 * p->head_dim * (p->dtype == PARROT_DTYPE_F32 ? 4.0 : 2.0), R = p->num_requests;
  const double owners = std::min(R, (double)T);            // requests that bring rows, at most
  const double prefixes = std::min((double)p->num_groups, owners * depth);
  const double own_mean = own * (R > 1 ? 0.55 : 1.0), pre_mean = pre * (prefixes > 1 ? 0.84 : 1.0);
  const double distinct = owners * own_mean + prefixes * pre_mean;   // tokens
  const double repeats = std::max(0.0, T * (own_mean + depth * pre_mean) - distinct);
  return 5.0 +
         std::max((depth * pre + own) * std::max(row, 512.0) / (wgs <= cus ? 74e3 : 42e3),
                  p->num_heads * row *
                      (distinct / 5.6e6 + repeats / (p->num_heads % 4 == 0 || p->num_heads <= 2 ? 28e6 : 12.5e6))) +
         1.45 * std::max(0.0, wgs / cus - 1.0);
}

parrot_status check_prefill(const parrot_problem* p, const parrot_prefill_rows* rows, bool nested,
                            PrefillPlan* pl) {
  if (!p) return fail(PARROT_ERR_INVALID_ARGUMENT, "problem is NULL");
  if (!rows) return fail(PARROT_ERR_INVALID_ARGUMENT, "rows is NULL");
  // the decode checks, with the group bound that prefill replaces by rows
  parrot_problem d = *p;
  if (d.num_groups > 0) d.max_group_size = d.num_requests > 0 ? 1 : d.max_group_size;
  parrot::Plan dpl;
  PARROT_TRY(check_problem(&d, &dpl));
  *pl = PrefillPlan{};
  const long T = rows->num_query_rows;
  if (T < 0) return fail(PARROT_ERR_INVALID_ARGUMENT, "num_query_rows %ld < 0", T);
  if (T == 0) return PARROT_OK;
  if (p->num_requests == 0) return fail(PARROT_ERR_INVALID_ARGUMENT, "num_query_rows %ld > 0 with no requests", T);
  const int mq = rows->max_query_rows;
  if (mq < 1 || mq > p->max_suffix_len)
    return fail(PARROT_ERR_INVALID_ARGUMENT, "max_query_rows %d not in [1, max_suffix_len = %d]", mq,
                p->max_suffix_len);
  if ((long)p->num_requests * mq < T)
    return fail(PARROT_ERR_INVALID_ARGUMENT, "num_query_rows %ld > num_requests * max_query_rows", T);
  const int mg = p->num_groups > 0 ? rows->max_group_rows : 0;
  if (mg < 0 || mg > T)
    return fail(PARROT_ERR_INVALID_ARGUMENT, "max_group_rows %d not in [0, num_query_rows]", mg);
  if (T * p->num_heads > 0x7fffffffL)
    return fail(PARROT_ERR_UNSUPPORTED, "num_query_rows * num_heads > 2^31 - 1");
  const int H = p->num_heads;
  pl->depth = p->num_groups > 0 ? (nested ? std::max(1, (int)p->max_prefix_depth) : 1) : 0;
  const int rows_per_tile = p->dtype == PARROT_DTYPE_F32 ? 64 : parrot::kWideRows;   // the kernel's tile height
  pl->qtiles_p = (int)ceil_div(mg, rows_per_tile);
  pl->qtiles_o = (int)ceil_div(mq, rows_per_tile);
  if (p->num_groups > 0 && pl->qtiles_p > 0) {
    pl->cp = prefill_chunk(p->max_prefix_len, (double)p->num_groups * H * pl->qtiles_p);
    pl->seg_p = (int)ceil_div(p->max_prefix_len, pl->cp);
  } else {
    pl->cp = kPrefillChunkMin;
    pl->seg_p = 0;
  }
  if (pl->seg_p > 0xFFFF)
    return fail(PARROT_ERR_UNSUPPORTED, "max_prefix_len %d needs %d prefix chunks (at most 65535)",
                p->max_prefix_len, pl->seg_p);
  pl->co = prefill_chunk(p->max_suffix_len, (double)p->num_requests * H * pl->qtiles_o);
  pl->seg_s = (int)ceil_div(p->max_suffix_len, pl->co);
  pl->seg_pre = pl->depth * pl->seg_p;
  pl->seg = pl->seg_pre + pl->seg_s;
  // work items per head (the grid holds them for every head, 8 heads apart
  // per XCD)
  pl->n_pre = (long)p->num_groups * pl->seg_p * pl->qtiles_p;
  pl->n_own = (long)p->num_requests * pl->seg_s * pl->qtiles_o;
  const int setting = single_pass_setting();
  const bool fits = p->max_prefix_len <= kPrefillChunkMax && p->max_suffix_len <= kPrefillChunkMax;
  const bool can = p->dtype != PARROT_DTYPE_F32 && !nested && fits;
  if (can && (setting == 1 || setting == 2)) {
    pl->kind = setting;
  } else if (setting == -1 || setting == 3) {
    // the tiled single-pass plans where they are expected to be faster (factors of
    // 0.93-0.95 lose no call of the sweeps by more than 3 %; 0.9 left 59 requests of
    // one row on split for 72 us, 61 stacked; 1.0 loses up to 1.21x)
    const PrefillCosts c = prefill_costs(p, rows, *pl);
    double best = c.split;
    if (can && setting == -1 && std::min(c.stacked, c.direct) < 0.95 * c.split) {
      best = std::min(c.stacked, c.direct);
      pl->kind = c.direct < c.stacked ? parrot::kPrefillDirect : parrot::kPrefillStacked;
    }
    const double one = direct_rows_cost(p, T, pl->depth);
    if (one >= 0.0 && (setting == 3 || one < (p->dtype == PARROT_DTYPE_F32 ? 1.45 : 0.6) * best)) {
      pl->kind = parrot::kPrefillRows;
      pl->waves = (double)T * H <= num_cus() ? 8 : 4;
    }
  }
  if (pl->kind != parrot::kPrefillSplit) {   // one item per group tile (whole prefix), one per own tile
    pl->n_pre = pl->kind == parrot::kPrefillStacked && pl->seg_p > 0 ? (long)p->num_groups * pl->qtiles_p : 0;
    pl->n_own = (long)p->num_requests * pl->qtiles_o;
  }
  const long grid = 8L * ceil_div(H, 8) * (pl->n_pre + pl->n_own);
  if (grid > 0x7fffffffL)
    return fail(PARROT_ERR_UNSUPPORTED, "prefill needs %ld workgroups (at most 2^31 - 1)", grid);
  const size_t n_slots = (size_t)T * H * pl->seg;
  auto align256 = [](size_t x) { return (x + 255) & ~(size_t)255; };
  pl->o_bytes = align256(n_slots * p->head_dim * sizeof(float));
  pl->lse_bytes = align256(n_slots * sizeof(float));
  pl->info_bytes = align256((size_t)T * parrot::kMetaInts * sizeof(int32_t));
  pl->total_bytes = pl->o_bytes + pl->lse_bytes + pl->info_bytes;
  return PARROT_OK;
}

parrot_status prefill(const parrot_problem* p, const parrot_prefill_rows* rows, const void* q,
                      const int32_t* qoff, const void* prefix_k, const void* prefix_v,
                      const void* suffix_k, const void* suffix_v, const int32_t* ptab,
                      const int32_t* plen, const int32_t* parents, const int32_t* stab,
                      const int32_t* slen, const int32_t* gid, void* out, float* lse,
                      void* workspace, size_t workspace_bytes, void* stream,
                      const parrot_trace* trace) {
  PrefillPlan pl;
  PARROT_TRY(check_prefill(p, rows, parents != nullptr, &pl));
  if (rows->num_query_rows == 0) {
    g_err.clear();
    return PARROT_OK;
  }
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const parrot_trace none = {nullptr, nullptr, nullptr, nullptr};
  const parrot_trace& tr = trace ? *trace : none;
  struct { const void* ptr; const char* name; size_t align; } req[] = {
      {q, "q", 16}, {qoff, "query_offsets", 4}, {suffix_k, "suffix_k", 16},
      {suffix_v, "suffix_v", 16}, {stab, "suffix_block_tables", 4}, {slen, "suffix_lens", 4},
      {gid, "group_ids", 4}, {out, "out", 16}, {lse, "lse", 4}, {workspace, "workspace", 256}};
  for (auto& r : req) {
    if (!r.ptr) return fail(PARROT_ERR_INVALID_ARGUMENT, "%s is NULL", r.name);
    if (!aligned(r.ptr, r.align)) return fail(PARROT_ERR_INVALID_ARGUMENT, "%s is not %zu-byte aligned", r.name, r.align);
  }
  if (p->num_groups > 0) {
    struct { const void* ptr; const char* name; size_t align; } preq[] = {
        {prefix_k, "prefix_k", 16}, {prefix_v, "prefix_v", 16},
        {ptab, "prefix_block_tables", 4}, {plen, "prefix_lens", 4}};
    for (auto& r : preq) {
      if (!r.ptr) return fail(PARROT_ERR_INVALID_ARGUMENT, "%s is NULL", r.name);
      if (!aligned(r.ptr, r.align)) return fail(PARROT_ERR_INVALID_ARGUMENT, "%s is not %zu-byte aligned", r.name, r.align);
    }
    if (parents && !aligned(parents, 4)) return fail(PARROT_ERR_INVALID_ARGUMENT, "prefix_parents is not 4-byte aligned");
  }
  if (workspace_bytes < pl.total_bytes)
    return fail(PARROT_ERR_WORKSPACE_TOO_SMALL, "workspace is %zu bytes, need %zu", workspace_bytes, pl.total_bytes);

  float* o_part = reinterpret_cast<float*>(workspace);
  float* lse_part = reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) + pl.o_bytes);
  int* merge_meta = reinterpret_cast<int*>(reinterpret_cast<char*>(workspace) + pl.o_bytes + pl.lse_bytes);
  const int T = rows->num_query_rows;
  if (pl.kind == parrot::kPrefillRows) {
    parrot::DirectArgs a{};
    a.q = q; a.pk = prefix_k; a.pv = prefix_v; a.sk = suffix_k; a.sv = suffix_v;
    a.ptab = ptab; a.plen = plen; a.stab = stab; a.slen = slen; a.gid = gid;
    a.parents = p->num_groups > 0 ? parents : nullptr; a.qoff = qoff;
    a.depth = std::max(1, pl.depth);
    a.out = out; a.lse = lse;
    a.R = p->num_requests; a.H = p->num_heads; a.NG = p->num_groups; a.T = T; a.max_q = rows->max_query_rows;
    a.pstride = p->prefix_table_stride; a.sstride = p->suffix_table_stride;
    a.max_p = p->max_prefix_len; a.max_s = p->max_suffix_len;
    a.npblk = p->num_groups > 0 ? p->num_prefix_blocks : 1; a.nsblk = p->num_suffix_blocks;
    a.scale_log2 = p->sm_scale * parrot::kLog2e;
    PARROT_TRY(launched(parrot::launch_direct(a, pl.waves, (int)p->dtype, p->head_dim, s, ev(tr.partials_start),
                                              ev(tr.partials_stop)),
                        "prefill kernel"));
    return no_merge(tr, s);
  }
  {
    parrot::PrefillArgs a{};
    a.q = q; a.pk = prefix_k; a.pv = prefix_v; a.sk = suffix_k; a.sv = suffix_v;
    a.ptab = ptab; a.plen = plen; a.stab = stab; a.slen = slen; a.gid = gid;
    a.parents = p->num_groups > 0 ? parents : nullptr; a.qoff = qoff;
    a.o_part = o_part; a.lse_part = lse_part; a.merge_meta = merge_meta;
    a.T = T; a.R = p->num_requests; a.H = p->num_heads; a.NG = p->num_groups;
    a.depth = std::max(1, pl.depth);
    a.pstride = p->prefix_table_stride; a.sstride = p->suffix_table_stride;
    a.max_p = p->max_prefix_len; a.max_s = p->max_suffix_len; a.max_q = rows->max_query_rows;
    a.npblk = p->num_groups > 0 ? p->num_prefix_blocks : 1; a.nsblk = p->num_suffix_blocks;
    a.seg = pl.seg; a.seg_p = pl.seg_p; a.seg_pre = pl.seg_pre; a.seg_s = pl.seg_s;
    a.cp = pl.cp; a.co = pl.co; a.qtiles_p = pl.qtiles_p; a.qtiles_o = pl.qtiles_o;
    a.n_pre = (int)pl.n_pre; a.n_own = (int)pl.n_own;
    a.meta_wgs = pl.kind != parrot::kPrefillSplit ? 0 : (T + 255) / 256;
    a.scale_log2 = p->sm_scale * parrot::kLog2e;
    a.plan = pl.kind;
    a.out = out; a.lse = lse;
    PARROT_TRY(launched(parrot::launch_prefill(a, (int)p->dtype, p->head_dim, s, ev(tr.partials_start),
                                               ev(tr.partials_stop)),
                        "prefill kernel"));
  }
  if (pl.kind != parrot::kPrefillSplit) return no_merge(tr, s);
  {
    parrot::MergeArgs a{};
    a.o_part = o_part; a.lse_part = lse_part; a.merge_meta = merge_meta;
    a.out = out; a.lse = lse;
    a.R = T; a.H = p->num_heads;
    a.seg = pl.seg; a.seg_p = pl.seg_p; a.seg_pre = pl.seg_pre;
    PARROT_TRY(launched(parrot::launch_merge(a, (int)p->dtype, p->head_dim, s, ev(tr.merge_start),
                                             ev(tr.merge_stop)),
                        "merge kernel"));
  }
  g_err.clear();
  return PARROT_OK;
}

}  // namespace

extern "C" {

size_t parrot_prefill_workspace_bytes(const parrot_problem* p, const parrot_prefill_rows* rows) {
  PrefillPlan pl;
  // sized for nested groups (depth max_prefix_depth): enough for flat calls too
  if (check_prefill(p, rows, true, &pl) != PARROT_OK) return (size_t)-1;
  g_err.clear();
  return pl.total_bytes;
}

int parrot_prefill_single_pass(const parrot_problem* p, const parrot_prefill_rows* rows, int nested) {
  PrefillPlan pl;
  if (check_prefill(p, rows, nested != 0, &pl) != PARROT_OK) return -1;
  g_err.clear();
  return pl.kind != parrot::kPrefillSplit ? 1 : 0;
}

// Test hook (not in parrot_attn.h): the plan a prefill takes (PrefillPlanKind; 16
// is added to kPrefillRows with eight waves per workgroup), -1 for invalid
// arguments.
int parrot_test_prefill_plan(const parrot_problem* p, const parrot_prefill_rows* rows, int nested) {
  PrefillPlan pl;
  if (check_prefill(p, rows, nested != 0, &pl) != PARROT_OK) return -1;
  return pl.kind + (pl.waves == 8 ? 16 : 0);
}

parrot_status parrot_shared_prefix_prefill(
    const parrot_problem* p, const parrot_prefill_rows* rows, const void* q,
    const int32_t* query_offsets, const void* prefix_k, const void* prefix_v,
    const void* suffix_k, const void* suffix_v, const int32_t* prefix_block_tables,
    const int32_t* prefix_lens, const int32_t* prefix_parents,
    const int32_t* suffix_block_tables, const int32_t* suffix_lens, const int32_t* group_ids,
    void* out, float* lse, void* workspace, size_t workspace_bytes, void* stream,
    const parrot_trace* trace) {
  return prefill(p, rows, q, query_offsets, prefix_k, prefix_v, suffix_k, suffix_v,
                 prefix_block_tables, prefix_lens, prefix_parents, suffix_block_tables,
                 suffix_lens, group_ids, out, lse, workspace, workspace_bytes, stream, trace);
}

}  // extern "C"

namespace {

parrot_status validate(const parrot_problem* p, const int32_t* prefix_block_tables,
                       const int32_t* prefix_lens, const int32_t* prefix_parents,
                       const int32_t* suffix_block_tables, const int32_t* suffix_lens,
                       const int32_t* group_ids, int32_t* scratch, void* stream,
                       const parrot_prefill_rows* rows = nullptr,
                       const int32_t* query_offsets = nullptr) {
  parrot::Plan pl;
  if (rows) {
    PrefillPlan fp;
    PARROT_TRY(check_prefill(p, rows, prefix_parents != nullptr, &fp));
    if (!query_offsets || !aligned(query_offsets, 4))
      return fail(PARROT_ERR_INVALID_ARGUMENT, "query_offsets is NULL or misaligned");
  } else {
    PARROT_TRY(check_problem(p, &pl));
  }
  if (p->num_requests == 0) { g_err.clear(); return PARROT_OK; }
  if (!scratch || !aligned(scratch, 4)) return fail(PARROT_ERR_INVALID_ARGUMENT, "scratch is NULL or misaligned");
  if (!suffix_block_tables || !suffix_lens || !group_ids)
    return fail(PARROT_ERR_INVALID_ARGUMENT, "suffix tables, suffix lengths and group ids are required");
  if (p->num_groups > 0 && (!prefix_block_tables || !prefix_lens))
    return fail(PARROT_ERR_INVALID_ARGUMENT, "prefix tables and lengths are required when num_groups > 0");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  hipError_t e = hipMemsetAsync(scratch, 0, 3 * sizeof(int32_t), s);
  if (e != hipSuccess) return fail(PARROT_ERR_HIP, "hipMemsetAsync: %s", hipGetErrorString(e));
  parrot::ValidateArgs a{};
  a.ptab = prefix_block_tables; a.plen = prefix_lens; a.stab = suffix_block_tables;
  a.slen = suffix_lens; a.gid = group_ids; a.result = scratch;
  a.parents = p->num_groups > 0 ? prefix_parents : nullptr;
  a.depth = std::max(1, (int)p->max_prefix_depth);
  a.R = p->num_requests; a.NG = p->num_groups; a.B = p->block_size;
  a.pstride = p->prefix_table_stride; a.sstride = p->suffix_table_stride;
  a.max_p = p->max_prefix_len; a.max_s = p->max_suffix_len;
  a.npblk = p->num_prefix_blocks; a.nsblk = p->num_suffix_blocks;
  if (rows) {
    a.qoff = query_offsets; a.T = rows->num_query_rows;
    a.max_q = rows->max_query_rows; a.max_grp = rows->max_group_rows;
  } else {
    a.max_grp = p->max_group_size;
  }
  PARROT_TRY(launched(parrot::launch_validate(a, s), "validation kernel"));
  int32_t res[3] = {0, 0, 0};
  e = hipMemcpyAsync(res, scratch, sizeof res, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail(PARROT_ERR_HIP, "reading validation result: %s", hipGetErrorString(e));
  static const char* what[] = {"", "group id out of [-1, num_groups)", "prefix length out of [1, max_prefix_len]",
                               "suffix length out of [0, max_suffix_len]", "empty context (prefix + suffix = 0)",
                               "prefix block id out of [0, num_prefix_blocks)",
                               "suffix block id out of [0, num_suffix_blocks)",
                               "prefix parent not in [-1, group)",
                               "prefix chain deeper than max_prefix_depth",
                               "query_offsets not 0 = offsets[0] <= ... <= offsets[R] = num_query_rows",
                               "query rows of a request > min(suffix length, max_query_rows)",
                               "rows reading a group's prefix > max_group_rows",
                               "requests reading a group's prefix > max_group_size"};
  constexpr int kCodes = (int)(sizeof what / sizeof what[0]) - 1;
  if (res[0] != 0)
    return fail(PARROT_ERR_INVALID_ARGUMENT, "%s at entry %d (value %d)",
                (res[0] > 0 && res[0] <= kCodes) ? what[res[0]] : "unknown", res[1], res[2]);
  g_err.clear();
  return PARROT_OK;
}

}  // namespace

extern "C" {

parrot_status parrot_validate_inputs(const parrot_problem* p, const int32_t* prefix_block_tables,
                                     const int32_t* prefix_lens, const int32_t* suffix_block_tables,
                                     const int32_t* suffix_lens, const int32_t* group_ids,
                                     int32_t* scratch, void* stream) {
  return validate(p, prefix_block_tables, prefix_lens, nullptr, suffix_block_tables, suffix_lens,
                  group_ids, scratch, stream);
}

parrot_status parrot_validate_nested_inputs(const parrot_problem* p, const int32_t* prefix_block_tables,
                                            const int32_t* prefix_lens, const int32_t* prefix_parents,
                                            const int32_t* suffix_block_tables,
                                            const int32_t* suffix_lens, const int32_t* group_ids,
                                            int32_t* scratch, void* stream) {
  if (p && p->num_requests > 0 && p->num_groups > 0 && !prefix_parents)
    return fail(PARROT_ERR_INVALID_ARGUMENT, "prefix_parents is NULL");
  return validate(p, prefix_block_tables, prefix_lens, prefix_parents, suffix_block_tables,
                  suffix_lens, group_ids, scratch, stream);
}

parrot_status parrot_validate_prefill_inputs(const parrot_problem* p, const parrot_prefill_rows* rows,
                                             const int32_t* query_offsets,
                                             const int32_t* prefix_block_tables,
                                             const int32_t* prefix_lens, const int32_t* prefix_parents,
                                             const int32_t* suffix_block_tables,
                                             const int32_t* suffix_lens, const int32_t* group_ids,
                                             int32_t* scratch, void* stream) {
  if (!rows) return fail(PARROT_ERR_INVALID_ARGUMENT, "rows is NULL");
  return validate(p, prefix_block_tables, prefix_lens, prefix_parents, suffix_block_tables,
                  suffix_lens, group_ids, scratch, stream, rows, query_offsets);
}

parrot_status parrot_hbm_read_ceiling(const void* src, size_t bytes, uint32_t* sink,
                                      int32_t workgroups, int32_t loads_per_thread,
                                      int32_t wave_spans, void* stream,
                                      const parrot_trace* trace) {
  if (!src || !sink) return fail(PARROT_ERR_INVALID_ARGUMENT, "src and sink must not be NULL");
  if (!aligned(src, 16) || !aligned(sink, 4))
    return fail(PARROT_ERR_INVALID_ARGUMENT, "src must be 16-byte and sink 4-byte aligned");
  if (bytes % 16 != 0) return fail(PARROT_ERR_INVALID_ARGUMENT, "bytes %zu is not a multiple of 16", bytes);
  if (workgroups < 1) return fail(PARROT_ERR_INVALID_ARGUMENT, "workgroups %d < 1", workgroups);
  if (loads_per_thread != 4 && loads_per_thread != 8 && loads_per_thread != 16)
    return fail(PARROT_ERR_UNSUPPORTED, "loads_per_thread %d (built for 4, 8 and 16)", loads_per_thread);
  if (wave_spans != 0 && wave_spans != 1)
    return fail(PARROT_ERR_INVALID_ARGUMENT, "wave_spans %d is not 0 or 1", wave_spans);
  PARROT_TRY(launched(parrot::launch_read_ceiling(src, bytes, sink, workgroups, loads_per_thread,
                                                  wave_spans != 0,
                                                  reinterpret_cast<hipStream_t>(stream),
                                                  trace ? ev(trace->partials_start) : nullptr,
                                                  trace ? ev(trace->partials_stop) : nullptr),
                      "read-ceiling kernel"));
  g_err.clear();
  return PARROT_OK;
}

parrot_status parrot_mfma_issue_ceiling(uint32_t* sink, int32_t workgroups, int32_t iters,
                                        int32_t valu_x4, void* stream, const parrot_trace* trace) {
  if (!sink) return fail(PARROT_ERR_INVALID_ARGUMENT, "sink must not be NULL");
  if (!aligned(sink, 4)) return fail(PARROT_ERR_INVALID_ARGUMENT, "sink must be 4-byte aligned");
  if (workgroups < 1) return fail(PARROT_ERR_INVALID_ARGUMENT, "workgroups %d < 1", workgroups);
  if (iters < 1) return fail(PARROT_ERR_INVALID_ARGUMENT, "iters %d < 1", iters);
  if (valu_x4 != 0 && valu_x4 != 8 && valu_x4 != 10 && valu_x4 != 11 && valu_x4 != 12 && valu_x4 != 16)
    return fail(PARROT_ERR_UNSUPPORTED, "valu_x4 %d (built for 0, 8, 10, 11, 12 and 16)", valu_x4);
  PARROT_TRY(launched(parrot::launch_mfma_issue(sink, workgroups, iters, valu_x4,
                                                reinterpret_cast<hipStream_t>(stream),
                                                trace ? ev(trace->partials_start) : nullptr,
                                                trace ? ev(trace->partials_stop) : nullptr),
                      "matrix-core issue kernel"));
  g_err.clear();
  return PARROT_OK;
}

const char* parrot_last_error(void) { return g_err.c_str(); }

int parrot_abi_version(void) { return PARROT_ABI_VERSION; }

}  // extern "C"
