// Small calls in one launch: one workgroup per (request, head) attends to the
// request's whole context and writes its output (decode), or one per (new row,
// head) of a prefill with few rows.
//
// The two-kernel path (partial results, merge) costs a small call two launches
// and about seven dependent memory round trips: lengths, scan, block table,
// K/V, partial results, descriptor, merge.  Here the waves of a workgroup share
// the request's blocks, every wave loads its own block-table entries (one per
// lane) beside the lengths, and the waves' results meet in LDS, which leaves
// lengths, group, K/V and the store.  Every request reads its group's prefix
// itself (repeats come from the caches; the workgroups of a head fall on one
// XCD when the heads are a multiple of 8), and nothing balances long contexts
// against short ones, so the host takes this path only where an estimate of
// both expects it to be faster (its rule carries the figures).
//
// Bound by round trips when the contexts are short (4.4 us a call, of which 3.4
// an empty launch), then by what one CU draws (about 75 KB/us per workgroup of
// eight waves from the caches, 50 from memory) and by the memory.  Measured, two
// kernels -> one: 4 fp32 requests of 150 tokens and 4 heads 9.0 -> 4.4 us; 7 chats
// of 40-700 tokens with append, 32 heads 16.6 -> 11.3; 8 requests of 300 tokens
// 15.3 -> 10.8.  Eight waves per workgroup up to one workgroup per CU, four above
// unless long contexts make eight faster (32 requests of 50 tokens: 11.3 us with
// eight, 9.6 with four; the chats 11.4 with eight, 13.2 with four; 9 requests of
// 50-900 tokens 15.1 and 15.9; sixteen waves are slower in the first two).
#include "common.h"

namespace parrot {

enum DirectMode { kDirectPlain = 0, kDirectAppend = 1, kDirectRows = 2 };

// NW: waves per workgroup.  MODE: plain decode, decode that appends this step's
// token, or prefill rows (a.qoff, a.T and a.max_q: workgroup (row, head), the
// row's request sees its prefixes and its own tokens up to the row's position).
template <int DT, int D, int MODE, int NW>
__global__ __launch_bounds__(NW * 64) void k_direct(DirectArgs a) {
  using E = Elem<DT>;
  constexpr bool APPEND = MODE == kDirectAppend;
  constexpr int ROW_B = D * E::kBytes;        // bytes per token row
  constexpr int LPT = ROW_B / 16;             // lanes per token
  constexpr int TPI = kWave / LPT;            // tokens per load instruction
  constexpr int IPB = kBlock / TPI;           // load instructions per block
  constexpr int EPL = E::kPerLoad;            // elements per lane load
  constexpr int BLK_B = kBlock * ROW_B;
  __shared__ float s_acc[NW][D];
  __shared__ float s_m[NW], s_l[NW];

  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int H = a.H;
  const int h = blockIdx.x % H;
  const int x = blockIdx.x / H;               // request, or prefill row
  int r = x;
  const int sub = lane % LPT;                 // which 16-byte slice of the row
  const int tg = lane / LPT;                  // token group
  const size_t blk_stride = (size_t)H * BLK_B;

  // one round of loads: the query, the lengths and the own table's entries.
  // Wave w takes blocks w, w + NW, ... of each list; lane k holds the entry of
  // its k-th (the host keeps every list within 64 NW blocks).
  const u32x4 q = ld16((const char*)a.q + ((size_t)(x * H + h) * D + sub * EPL) * E::kBytes);
  const int col = w + NW * lane;
  int first = 0, count = 0;
  if constexpr (MODE == kDirectRows) {
    // the row's request: the last one whose first row is at or before it.  The
    // lanes test every step-th request, then the requests of that step: a round
    // trip per factor of 64 (8 rows of the last of 4096 requests, 8 heads: 6.1 us;
    // walked 64 at a time 16.2).
    r = -1;
    for (int base = 0, n = a.R; n > 0;) {
      const int step = (n + kWave - 1) / kWave;
      const int at = lane * step;
      const int k = __popcll(__ballot(at < n && a.qoff[base + min(at, n - 1)] <= x));
      if (k == 0 || step == 1) { r = base + k - 1; break; }
      base += (k - 1) * step;
      n = min(step, n - (k - 1) * step);
    }
    first = r >= 0 ? clampi(a.qoff[r], 0, a.T) : 0;
    const long n = r >= 0 ? (long)a.qoff[r + 1] - a.qoff[r] : 0;
    count = (int)(n < 0 ? 0 : n > a.max_q ? a.max_q : n);
    r = r < 0 ? 0 : r;
  }
  int e_own = 0;
  if (a.sstride > 0) e_own = a.stab[(long)r * a.sstride + min(col, a.sstride - 1)];
  int S = clampi(a.slen[r], 0, a.max_s);
  int g = a.gid[r];
  if constexpr (MODE == kDirectRows) {
    // own tokens up to the row's position; a row that no request holds (as
    // when a request has more rows than the bounds allow) sees nothing
    count = min(count, min(S, a.T - first));
    const int pos = S - count + (x - first);
    const bool held = x >= first && x < first + count;
    S = held ? pos + 1 : 0;
    g = held ? g : -1;
  }
  const int nbs = (S + kBlock - 1) / kBlock;

  // the prefixes of the request's chain of groups, innermost first
  int e_pre[kMaxDepth], plen[kMaxDepth];
#pragma unroll
  for (int l = 0; l < kMaxDepth; ++l) {
    e_pre[l] = 0; plen[l] = 0;
    if (l < a.depth && g >= 0 && g < a.NG) {
      e_pre[l] = a.ptab[(long)g * a.pstride + min(col, a.pstride - 1)];
      plen[l] = clampi(a.plen[g], 0, a.max_p);
      g = a.parents ? a.parents[g] : -1;
    } else {
      g = -1;
    }
  }

  // the wave's blocks: own tokens, then the levels
  auto mine = [&](int nb) { return nb > w ? (nb - w + NW - 1) / NW : 0; };
  int end[kMaxDepth + 1];
  end[0] = mine(nbs);
#pragma unroll
  for (int l = 0; l < kMaxDepth; ++l)
    end[l + 1] = end[l] + mine((plen[l] + kBlock - 1) / kBlock);
  const int total = end[kMaxDepth];

  struct Blk {
    u32x4 k[IPB], v[IPB];
    int ntok;        // valid tokens
    int app;         // APPEND: load holding this lane's share of the new token, else -1
    size_t app_off;  // APPEND: its pool byte offset
  };
  auto fetch = [&](Blk& B, int t) {
    const char* kp = (const char*)a.sk;
    const char* vp = (const char*)a.sv;
    int nblk = a.nsblk;
    int i = t, entry = __builtin_amdgcn_readlane(e_own, t & 63);
    int len = S;
    bool own = true;
#pragma unroll
    for (int l = 0; l < kMaxDepth; ++l) {
      if (t >= end[l]) {                       // wave-uniform
        own = false;
        i = t - end[l];
        entry = __builtin_amdgcn_readlane(e_pre[l], i & 63);
        len = plen[l];
        kp = (const char*)a.pk; vp = (const char*)a.pv; nblk = a.npblk;
      }
    }
    const int j = w + NW * i;                  // block of its list
    const int blk = clampi(entry, 0, nblk - 1);
    const size_t off = blk * blk_stride + (size_t)h * BLK_B + (size_t)lane * 16;
    const int ntok = len - j * kBlock;
    B.ntok = ntok < kBlock ? ntok : kBlock;
    if constexpr (APPEND) {
      // the own tokens' last block holds the new token at slot (S - 1) % 16
      B.app = -1;
      if (own && j == nbs - 1) {
        const int last = (S - 1) % kBlock;
        if (tg == last % TPI) B.app = last / TPI;
      }
      B.app_off = off + (size_t)(B.app < 0 ? 0 : B.app) * 1024;
      const size_t noff = (size_t)(r * H + h) * D * E::kBytes + (size_t)sub * 16;
#pragma unroll
      for (int n = 0; n < IPB; ++n) {
        const bool nw = n == B.app;
        B.k[n] = ld16(nw ? (const char*)a.k_new + noff : kp + off + n * 1024);
        B.v[n] = ld16(nw ? (const char*)a.v_new + noff : vp + off + n * 1024);
      }
    } else {
#pragma unroll
      for (int n = 0; n < IPB; ++n) {
        B.k[n] = ld16(kp + off + n * 1024);
        B.v[n] = ld16(vp + off + n * 1024);
      }
    }
  };

  float m = -INFINITY, l = 0.f;
  float acc[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
  auto reduce = [&](Blk& B) {
    if constexpr (APPEND) {
#pragma unroll
      for (int n = 0; n < IPB; ++n)
        if (n == B.app) {                      // write this step's token into the cache
          *reinterpret_cast<u32x4*>((char*)a.app_k + B.app_off) = B.k[n];
          *reinterpret_cast<u32x4*>((char*)a.app_v + B.app_off) = B.v[n];
        }
    }
    float s[IPB];
#pragma unroll
    for (int n = 0; n < IPB; ++n) s[n] = group_sum<LPT>(E::dot(B.k[n], q)) * a.scale_log2;
    if (B.ntok < kBlock) {                     // partly filled block: mask the tail
#pragma unroll
      for (int n = 0; n < IPB; ++n)
        if (n * TPI + tg >= B.ntok) {
          s[n] = -INFINITY;
          B.v[n] = u32x4{0u, 0u, 0u, 0u};      // 0 * NaN would poison the sum
        }
    }
    float bm = s[0];
#pragma unroll
    for (int n = 1; n < IPB; ++n) bm = fmaxf(bm, s[n]);
    const float mn = fmaxf(m, bm);
    const float mref = (mn == -INFINITY) ? 0.f : mn;
    const float alpha = fast_exp2(m - mref);
    float p[IPB], psum = 0.f;
#pragma unroll
    for (int n = 0; n < IPB; ++n) { p[n] = fast_exp2(s[n] - mref); psum += p[n]; }
    l = l * alpha + psum;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] *= alpha;
#pragma unroll
    for (int n = 0; n < IPB; ++n) {
      float v[EPL];
      E::to_f32(B.v[n], v);
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[e] = __builtin_fmaf(p[n], v[e], acc[e]);
    }
    m = mn;
  };

  // one block is reduced while the next one's loads are in flight (not where a
  // block takes 64 registers).  Deeper rings were slower: the repeated loads
  // past the end that keep them branch-free cost more than they hide.
  if constexpr (IPB > 4) {
    for (int t = 0; t < total; ++t) {
      Blk A;
      fetch(A, t);
      reduce(A);
    }
  } else if (total > 0) {
    Blk A, B;
    fetch(A, 0);
    for (int t = 0;; t += 2) {
      if (t + 1 >= total) { reduce(A); break; }
      fetch(B, t + 1);
      reduce(A);
      if (t + 2 >= total) { reduce(B); break; }
      fetch(A, t + 2);
      reduce(B);
    }
  }
  // the wave's token groups, then the waves
#pragma unroll
  for (int off = LPT; off < kWave; off <<= 1) {
    const float mo = __shfl_xor(m, off), lo = __shfl_xor(l, off);
    const float mn = fmaxf(m, mo);
    const float mref = (mn == -INFINITY) ? 0.f : mn;
    const float sa = fast_exp2(m - mref), sb = fast_exp2(mo - mref);
    l = l * sa + lo * sb;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = acc[e] * sa + __shfl_xor(acc[e], off) * sb;
    m = mn;
  }
  if (tg == 0) {
#pragma unroll
    for (int e = 0; e < EPL; e += 4)
      *reinterpret_cast<f32x4*>(&s_acc[w][sub * EPL + e]) = f32x4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
    if (lane == 0) { s_m[w] = m; s_l[w] = l; }
  }
  __syncthreads();
  const int d = threadIdx.x;
  if (d >= D) return;
  float mx = s_m[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) mx = fmaxf(mx, s_m[i]);
  // (no guard on mx: as in the merge, logits that are all -inf give NaN)
  float tot = 0.f, o = 0.f;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const float c = fast_exp2(s_m[i] - mx);
    tot = __builtin_fmaf(c, s_l[i], tot);
    o = __builtin_fmaf(c, s_acc[i][d], o);
  }
  // an empty context is defined as out = 0, lse = -inf; it is told by its length,
  // since a sum that is not positive can also come from NaN or infinite inputs,
  // which have to reach the output
  bool empty = S <= 0;
#pragma unroll
  for (int l = 0; l < kMaxDepth; ++l) empty = empty && plen[l] <= 0;
  E::store1((char*)a.out + ((size_t)(x * H + h) * D + d) * E::kBytes, empty ? 0.f : o / tot);
  if (d == 0) a.lse[x * H + h] = empty ? -INFINITY : (mx + fast_log2(tot)) * kLn2;
}

template <int DT, int D, int NW>
static void launch_direct_nw(const DirectArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid((unsigned)((a.qoff ? a.T : a.R) * a.H)), wg(NW * 64);
  if (a.qoff)
    hipExtLaunchKernelGGL((k_direct<DT, D, kDirectRows, NW>), grid, wg, 0, s, e0, e1, 0, a);
  else if (a.k_new)
    hipExtLaunchKernelGGL((k_direct<DT, D, kDirectAppend, NW>), grid, wg, 0, s, e0, e1, 0, a);
  else
    hipExtLaunchKernelGGL((k_direct<DT, D, kDirectPlain, NW>), grid, wg, 0, s, e0, e1, 0, a);
}

template <int DT, int D>
static hipError_t launch_direct_t(const DirectArgs& a, int waves, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (waves == 8)
    launch_direct_nw<DT, D, 8>(a, s, e0, e1);
  else
    launch_direct_nw<DT, D, 4>(a, s, e0, e1);
  return hipGetLastError();
}

hipError_t launch_direct(const DirectArgs& a, int waves, int dtype, int D, hipStream_t s, hipEvent_t e0,
                         hipEvent_t e1) {
  // a lane holds one table entry per list: at most 64 blocks per wave and list
  const int most = waves * kWave * kBlock;
  const long groups = (long)(a.qoff ? a.T : a.R) * a.H;
  if (a.R < 1 || a.H < 1 || groups < 1 || groups > kDirectMaxWgs || a.depth > kMaxDepth ||
      (waves != 4 && waves != 8) || a.max_s > most || (a.NG > 0 && a.max_p > most) || (a.qoff && a.k_new))
    return hipErrorInvalidValue;
  switch (dtype * 1000 + D) {
    case kF32 * 1000 + 64: return launch_direct_t<kF32, 64>(a, waves, s, e0, e1);
    case kF32 * 1000 + 128: return launch_direct_t<kF32, 128>(a, waves, s, e0, e1);
    case kF16 * 1000 + 64: return launch_direct_t<kF16, 64>(a, waves, s, e0, e1);
    case kF16 * 1000 + 128: return launch_direct_t<kF16, 128>(a, waves, s, e0, e1);
    case kBF16 * 1000 + 64: return launch_direct_t<kBF16, 64>(a, waves, s, e0, e1);
    case kBF16 * 1000 + 128: return launch_direct_t<kBF16, 128>(a, waves, s, e0, e1);
  }
  return hipErrorInvalidValue;
}

}  // namespace parrot
