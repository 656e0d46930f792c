// Split-KV decode attention over paged K/V: the non-shared tokens of every
// request (and, on the per-request path, its group's prefix as well).
//
// Work layout.  Each request owns a row of 16-token block columns (its own
// tokens; on the per-request path its group's prefix blocks first).  The rows
// are laid end to end into one flat column list, which is cut into equal runs
// of Q columns ("column groups").  Wave (g, h) reduces head h over column
// group g, so every wave streams the same number of bytes, and the H waves of
// a group walk the same physical blocks at the same time, reading all heads
// of a 16-token block (one contiguous region of H token blocks per tensor)
// together.  With HPW = 2 a wave reduces the adjacent heads h, h + 1 (H / 2
// waves per group): one contiguous piece of two heads per block and tensor.
// The role's grid is a fixed number of 4-wave workgroups per CU, so the
// per-CU load is even too.  A run
// may cross request boundaries: the wave then emits one partial result
// (normalised output and base-2 log-sum-exp) per (request, head) piece.
//
// Per block, a token row is D*elt bytes read as D*elt/16 lanes x 16 bytes, so
// each load instruction covers a contiguous 1 KiB of the block (coalesced
// 128-bit loads).  Each group of lanes that shares a token computes its slice
// of q.k, the slices are summed with DPP row operations, and every token group
// keeps its own online-softmax state; the groups are combined at the end of a
// piece.  One block is reduced while the next one's loads are in flight (not on
// most fp32 paths, see the loop); the loop is unrolled by two with ping-pong
// registers and every load inside it is unconditional, so the compiler's
// memory-wait counts stay exact.
#pragma once
#include <type_traits>

#include "common.h"

namespace parrot {

#ifndef PARROT_SPLITKV_STREAM_SCALAR_TABLE
#define PARROT_SPLITKV_STREAM_SCALAR_TABLE 0
#endif
// Streaming path: block-table entries as scalar loads (the next block's loads
// then issue while the current block is in flight) instead of vector loads.
constexpr bool kStreamScalarTable = PARROT_SPLITKV_STREAM_SCALAR_TABLE != 0;

// LDS bytes the split-KV role needs: two per-request arrays (six on the
// per-request path) and a total per wave.
constexpr int kSplitkvLds = (2 * kMaxRequests + kSkvWaves) * 4;
static_assert((6 * kMaxRequestsPrefix + kSkvWaves) * 4 <= kSplitkvLds, "the per-request path's arrays fit");
static_assert(kMaxRequests <= kWave * kWave, "two probes find a column's request");

// Inclusive sum over the wave's lanes (DPP row shifts, then row broadcasts).
PARROT_DEV int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);   // row_shr 1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);   // row_shr 2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);   // row_shr 4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);   // row_shr 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);   // row_bcast 15 into rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);   // row_bcast 31 into rows 2, 3
  return x;
}

// One workgroup of the split-KV role; `wg` is the role-local workgroup index
// and a.nwaves = 4 x (number of split-KV workgroups).
//
// Load policy, chosen per path by measurement on MI355X:
//  * STREAM (the shared path: every KV block is read once per call): K/V use
//    a nontemporal hint, and a block's table entry is an ordinary vector
//    load.  Waiting for that entry also waits for the previous block, so
//    about one block per wave is in flight; with the HBM already saturated
//    this runs slightly faster than keeping two blocks in flight.
//  * per-request path (each member re-reads its group's prefix, mostly from
//    the caches): cached K/V loads, and table entries as scalar loads so the
//    next block's K/V loads can issue while the current block is in flight.
//
// APPEND: the last own token of every request with S_r >= 1 is this decode
// step's token.  Its K/V are taken from k_new / v_new instead of the pool, and
// the lanes that hold it write it into the pool slot (stab[r][(S_r-1)/16],
// (S_r-1)%16) while the block is reduced, so the cache holds it for later
// steps.  The lane that writes a 16-byte piece is the lane that would have
// read it, and no other wave reads that (block, head) in the call.
template <int DT, int D, bool STREAM, bool APPEND = false, int HPW = 1>
__device__ __forceinline__ void splitkv_role(const SplitKVArgs& a, char* lds, int wg) {
  static_assert(HPW == 1 || HPW == 2, "one or two heads per wave");
  using E = Elem<DT>;
  constexpr int ROW_B = D * E::kBytes;        // bytes per token row
  constexpr int LPT = ROW_B / 16;             // lanes per token
  constexpr int TPI = kWave / LPT;            // tokens per load instruction
  constexpr int IPB = kBlock / TPI;           // load instructions per block
  constexpr int EPL = E::kPerLoad;            // elements per lane load
  constexpr int BLK_B = kBlock * ROW_B;
  static_assert(TPI * ROW_B == 1024, "one instruction covers 1 KiB");

  // per-request data: first flat block per head-sequence, own token counts and,
  // on the per-request path, blocks per sequence, leading prefix blocks, group
  // and prefix tokens
  constexpr int MAXR = STREAM ? kMaxRequests : kMaxRequestsPrefix;
  int* s_excl = reinterpret_cast<int*>(lds);
  int* s_slen = s_excl + MAXR;
  int* s_tot = s_slen + MAXR;                 // columns per scanning wave
  int* s_cnt = s_tot + kSkvWaves;             // per-request path only from here on
  int* s_nbp = s_cnt + MAXR;
  int* s_g = s_nbp + MAXR;
  int* s_plen = s_g + MAXR;

  const int lane = threadIdx.x & 63;
  const int wave_in_wg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int R = a.R, H = a.H;

  {
    // Wave v scans requests [v * per, (v + 1) * per): their own lengths (and, on
    // the per-request path, groups and prefix lengths) are all loaded before the
    // scan, one memory round trip (two on the per-request path) whatever R.
    // Addresses are clamped into [0, R).  One wave scanning 1024 requests with
    // shuffles through the LDS, and a second launch above 1024, cost 1000
    // requests of 50 tokens (8 heads) 52.7 us against 48.3, 1500 requests in 24
    // groups 370 us against 331 and 4000 of them 552 against 376 (member scan of
    // the prefix role included).
    // Up to 256 requests take one step per wave, built without the others' tests
    // (8 requests of 50-300 tokens on a 2000-token prefix 18.0 -> 17.4 us, 200 on
    // 700 40.2 -> 39.5).
    auto scan = [&](auto steps) {
      constexpr int kIt = decltype(steps)::value;
      const int it = kIt == 1 ? 1 : (R + kWave * kSkvWaves - 1) / (kWave * kSkvWaves);   // 64-request steps per wave, <= kIt
      const int r0 = wave_in_wg * it * kWave;
      int s_in[kIt], g_in[STREAM ? 1 : kIt], p_in[STREAM ? 1 : kIt];
#pragma unroll
      for (int i = 0; i < kIt; ++i) s_in[i] = i < it ? a.slen[min(r0 + i * kWave + lane, R - 1)] : 0;
      if constexpr (!STREAM) {
#pragma unroll
        for (int i = 0; i < kIt; ++i) {
          const int g = a.gid[min(r0 + i * kWave + lane, R - 1)];
          g_in[i] = (g >= 0 && g < a.NG) ? g : -1;
          p_in[i] = 0;
        }
        if (a.NG > 0) {                          // no prefix lengths exist without groups
#pragma unroll
          for (int i = 0; i < kIt; ++i) p_in[i] = a.plen[g_in[i] >= 0 ? g_in[i] : 0];
        }
      }
      int carry = 0;
      int excl[kIt];
#pragma unroll
      for (int i = 0; i < kIt; ++i) {
        excl[i] = 0;
        if (i < it) {                            // wave-uniform
          const int r = r0 + i * kWave + lane;
          const bool valid = r < R;
          const int S = valid ? clampi(s_in[i], 0, a.max_s) : 0;
          int cnt = (S + kBlock - 1) / kBlock;
          if (valid) s_slen[r] = S;
          if constexpr (!STREAM) {
            const int g = valid ? g_in[i] : -1;
            const int P = g >= 0 ? clampi(p_in[i], 0, a.max_p) : 0;
            const int nbp = (P + kBlock - 1) / kBlock;
            cnt += nbp;
            if (valid) { s_cnt[r] = cnt; s_nbp[r] = nbp; s_g[r] = g; s_plen[r] = P; }
          }
          const int incl = wave_scan(cnt);
          excl[i] = carry + incl - cnt;
          if (valid) s_excl[r] = excl[i];
          carry += __builtin_amdgcn_readlane(incl, kWave - 1);
        }
      }
      if (lane == 0) s_tot[wave_in_wg] = carry;
      __syncthreads();
      if (R > kWave) {                           // else wave 0 scanned them all
        int before = 0;
#pragma unroll
        for (int v = 0; v < kSkvWaves - 1; ++v) before += v < wave_in_wg ? s_tot[v] : 0;
#pragma unroll
        for (int i = 0; i < kIt; ++i) {
          const int r = r0 + i * kWave + lane;
          if (i < it && r < R) s_excl[r] = before + excl[i];
        }
        __syncthreads();
      }
    };
    if (R <= kWave * kSkvWaves)
      scan(std::integral_constant<int, 1>{});
    else
      scan(std::integral_constant<int, MAXR / kWave / kSkvWaves>{});
  }
  int s_total = 0;
#pragma unroll
  for (int v = 0; v < kSkvWaves; ++v) s_total += s_tot[v];
  // block columns of request r's sequence
  auto cols = [&](int r) { return STREAM ? (s_slen[r] + kBlock - 1) / kBlock : s_cnt[r]; };
  const int C = s_total;                                      // flat block columns
  const int HG = H / HPW;                                     // head groups (H % HPW == 0)
  const int G = a.nwaves / HG;                                // column groups
  const int Qg = (C + G - 1) / G;
  const int Q = Qg > a.min_q ? Qg : a.min_q;                  // columns per group
  if (wg == 0) {
    // Merge descriptor of each request: how many prefix-chunk slots (shared
    // path: chunks of its group's prefix) and how many split-KV pieces (the
    // column groups its run of columns touches) hold its partial results.
    // With nested groups, the request's chain is walked from its own group
    // outwards (at most depth groups); level l counts from the outermost.
    for (int rr = threadIdx.x; rr < R; rr += blockDim.x) {
      int np[kMaxDepth] = {0, 0, 0, 0};
      int nlev = 0;
      if (!a.with_prefix) {
        int chain[kMaxDepth];
        int x = a.gid[rr];
        while (x >= 0 && x < a.NG && nlev < a.depth) {
          chain[nlev++] = x;
          x = a.parents ? a.parents[x] : -1;
        }
#pragma unroll
        for (int i = 0; i < kMaxDepth; ++i)
          if (i < nlev) np[nlev - 1 - i] = (clampi(a.plen[chain[i]], 0, a.max_p) + a.cp - 1) / a.cp;
      }
      const int first = s_excl[rr], n = cols(rr);
      const int ns = n > 0 ? (first + n - 1) / Q - first / Q + 1 : 0;
      *reinterpret_cast<int4*>(a.merge_meta + kMetaInts * rr) =
          make_int4(ns, nlev, (int)((unsigned)np[0] | ((unsigned)np[1] << 16)),
                    (int)((unsigned)np[2] | ((unsigned)np[3] << 16)));
    }
  }
  const int w = wg * kSkvWaves + wave_in_wg;
  const int grp = w / HG;
  const int h = (w % HG) * HPW;               // first head of the wave (HPW adjacent heads)
  const int c0 = grp * Q;
  if (grp >= G || c0 >= C) return;
  const int nblk_run = (C - c0 < Q) ? (C - c0) : Q;

  // the request holding column c0: the last request whose first column is <= c0
  // (lanes test every step-th request, then the requests of that step)
  const int step = (R + kWave - 1) / kWave;                   // <= 64
  const int probe = lane * step;
  const int seg0 = (__popcll(__ballot(probe < R && s_excl[min(probe, R - 1)] <= c0)) - 1) * step;
  const int cand = seg0 + lane;
  int r = seg0;
  if (step > 1)
    r += __popcll(__ballot(lane < step && cand < R && s_excl[clampi(cand, 0, R - 1)] <= c0)) - 1;
  r = clampi(r, 0, R - 1);                                    // in range whatever the data
  int cnt = cols(r);
  if (cnt <= 0) return;                       // unreachable for consistent data
  int b = c0 - s_excl[r];

  const int sub = lane % LPT;                 // which 16-byte slice of the row
  const int tg = lane / LPT;                  // token group
  const size_t blk_stride = (size_t)H * BLK_B;

  // One fetched block: K and V slices of the wave's heads (adjacent in the
  // pool, so HPW * 4 KiB contiguous per tensor), the matching query slices,
  // and the metadata needed to reduce it and to close its piece.
  struct Blk {
    u32x4 k[HPW * IPB], v[HPW * IPB], q[HPW];
    int ntok;      // valid tokens in the block
    int seq;       // r * H + h (first head)
    int piece_end; // last block of its sequence
    int app;       // APPEND: piece (of a head's IPB loads) holding this lane's share of the new token, else -1
    size_t app_off;  // APPEND: pool byte offset of that piece for the first head
  };
  auto fetch = [&](Blk& B) {
    const int nbp = STREAM ? 0 : s_nbp[r];
    const char* kp;
    const char* vp;
    int entry, nblk, ntok;
    if (!STREAM && b < nbp) {
      entry = (STREAM && !kStreamScalarTable) ? a.ptab[(long)s_g[r] * a.pstride + b]
                                              : ld_uniform(a.ptab + (long)s_g[r] * a.pstride + b);
      kp = (const char*)a.pk; vp = (const char*)a.pv; nblk = a.npblk;
      ntok = s_plen[r] - b * kBlock;
    } else {
      const int bs = b - nbp;
      entry = (STREAM && !kStreamScalarTable) ? a.stab[(long)r * a.sstride + bs]
                                              : ld_uniform(a.stab + (long)r * a.sstride + bs);
      kp = (const char*)a.sk; vp = (const char*)a.sv; nblk = a.nsblk;
      ntok = s_slen[r] - bs * kBlock;
    }
    const int blk = clampi(entry, 0, nblk - 1);
    const size_t off = blk * blk_stride + (size_t)h * BLK_B + (size_t)lane * 16;
    if constexpr (APPEND) {
      // the own tokens' last block holds the new token at slot (S - 1) % 16
      B.app = -1;
      if (b >= nbp && b == cnt - 1) {
        const int last = (s_slen[r] - 1) % kBlock;
        if (tg == last % TPI) B.app = last / TPI;
      }
      B.app_off = off + (size_t)(B.app < 0 ? 0 : B.app) * 1024;   // first head's piece
#pragma unroll
      for (int i = 0; i < HPW * IPB; ++i) {
        // load i is piece i % IPB of head h + i / IPB; the new token's pieces
        // come from k_new / v_new
        const size_t noff = ((size_t)(r * H + h + i / IPB) * D) * E::kBytes + (size_t)sub * 16;
        const bool nw = (i % IPB) == B.app;
        const char* ks = nw ? (const char*)a.k_new + noff : kp + off + i * 1024;
        const char* vs = nw ? (const char*)a.v_new + noff : vp + off + i * 1024;
        B.k[i] = STREAM ? ld16_stream(ks) : ld16(ks);
        B.v[i] = STREAM ? ld16_stream(vs) : ld16(vs);
      }
    } else {
#pragma unroll
      for (int i = 0; i < HPW * IPB; ++i) {
        B.k[i] = STREAM ? ld16_stream(kp + off + i * 1024) : ld16(kp + off + i * 1024);
        B.v[i] = STREAM ? ld16_stream(vp + off + i * 1024) : ld16(vp + off + i * 1024);
      }
    }
#pragma unroll
    for (int u = 0; u < HPW; ++u)
      B.q[u] = ld16((const char*)a.q + ((size_t)(r * H + h + u) * D + sub * EPL) * E::kBytes);
    B.ntok = ntok < kBlock ? ntok : kBlock;
    B.seq = r * H + h;
    B.piece_end = (b == cnt - 1);
    // advance the cursor to the next column (same head)
    if (++b == cnt) {
      b = 0;
      do { ++r; } while (r < R && cols(r) == 0);
      cnt = r < R ? cols(r) : 1;
    }
  };

  float m[HPW], l[HPW];
  float acc[HPW][EPL];
#pragma unroll
  for (int u = 0; u < HPW; ++u) {
    m[u] = -INFINITY; l[u] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[u][e] = 0.f;
  }

  // close the current piece of sequences seq .. seq + HPW - 1 (the wave's
  // heads): combine the token groups, write the normalised output and
  // log-sum-exp, reset the state
  auto close_piece = [&](int seq) {
    const int piece = grp - s_excl[seq / H] / Q;
#pragma unroll
    for (int u = 0; u < HPW; ++u) {
#pragma unroll
      for (int off = LPT; off < kWave; off <<= 1) {
        const float mo = __shfl_xor(m[u], off);
        const float lo = __shfl_xor(l[u], off);
        const float mn = fmaxf(m[u], mo);
        const float mref = (mn == -INFINITY) ? 0.f : mn;
        const float sa = fast_exp2(m[u] - mref), sb = fast_exp2(mo - mref);
        l[u] = l[u] * sa + lo * sb;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[u][e] = acc[u][e] * sa + __shfl_xor(acc[u][e], off) * sb;
        m[u] = mn;
      }
      if (tg == 0) {
        const size_t slot = (size_t)(seq + u) * a.seg + a.seg_pre + piece;
        const float inv = 1.f / l[u];
        float* o = a.o_part + slot * D + sub * EPL;
#pragma unroll
        for (int e = 0; e < EPL; e += 4)
          *reinterpret_cast<f32x4*>(o + e) = f32x4{acc[u][e] * inv, acc[u][e + 1] * inv,
                                                   acc[u][e + 2] * inv, acc[u][e + 3] * inv};
        if (lane == 0) a.lse_part[slot] = m[u] + fast_log2(l[u]);
      }
      m[u] = -INFINITY; l[u] = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[u][e] = 0.f;
    }
  };

  auto reduce = [&](Blk& B, bool run_end) {
    if constexpr (APPEND) {
      if (B.app >= 0) {                        // write this step's token into the cache
#pragma unroll
        for (int u = 0; u < HPW; ++u)
#pragma unroll
          for (int i = 0; i < IPB; ++i) {
            if (i == B.app) {
              const size_t wo = B.app_off + (size_t)u * BLK_B;       // head h + u
              *reinterpret_cast<u32x4*>((char*)a.app_k + wo) = B.k[u * IPB + i];
              *reinterpret_cast<u32x4*>((char*)a.app_v + wo) = B.v[u * IPB + i];
            }
          }
      }
    }
#pragma unroll
    for (int u = 0; u < HPW; ++u) {
      u32x4* bk = B.k + u * IPB;
      u32x4* bv = B.v + u * IPB;
      float s[IPB];
#pragma unroll
      for (int i = 0; i < IPB; ++i) s[i] = group_sum<LPT>(E::dot(bk[i], B.q[u])) * a.scale_log2;
      if (B.ntok < kBlock) {                  // partly filled block: mask the tail
#pragma unroll
        for (int i = 0; i < IPB; ++i) {
          if (i * TPI + tg >= B.ntok) {
            s[i] = -INFINITY;
            bv[i] = u32x4{0u, 0u, 0u, 0u};    // 0 * NaN would poison the sum
          }
        }
      }
      float bm = s[0];
#pragma unroll
      for (int i = 1; i < IPB; ++i) bm = fmaxf(bm, s[i]);
      const float mn = fmaxf(m[u], bm);
      const float mref = (mn == -INFINITY) ? 0.f : mn;
      const float alpha = fast_exp2(m[u] - mref);
      float psum = 0.f;
      float p[IPB];
#pragma unroll
      for (int i = 0; i < IPB; ++i) { p[i] = fast_exp2(s[i] - mref); psum += p[i]; }
      l[u] = l[u] * alpha + psum;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[u][e] *= alpha;
#pragma unroll
      for (int i = 0; i < IPB; ++i) {
        float v[EPL];
        E::to_f32(bv[i], v);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[u][e] = __builtin_fmaf(p[i], v[e], acc[u][e]);
      }
      m[u] = mn;
    }
    if (B.piece_end || run_end) close_piece(B.seq);
  };

  // A block of an fp32 cache is 64 registers (128-wide heads) or 32: two of them
  // in ping-pong spilled to scratch at 128 (112 registers, some of them stored
  // and reloaded for every block) and at 64 the streaming loop was slower too,
  // so those run block by block.  On MI355X, ping-pong -> block by block:
  // 128-wide, 200 requests of 10-300 own tokens on 300, 8 heads 84 -> 61 us, 80 of
  // 300-900 on 600 108 -> 72, read per request 196 -> 97; 64-wide, the same two
  // calls 37.6 -> 32.7 and 41.7 -> 38.9.  The per-request path keeps ping-pong at
  // 64 (cached loads with scalar table entries keep two blocks in flight; 44.6 us
  // block by block, 43.2 in ping-pong).
  if constexpr (DT == kF32 && (STREAM || IPB > 4)) {
    for (int i = 0; i < nblk_run; ++i) {
      Blk A;
      fetch(A);
      reduce(A, i + 1 == nblk_run);
    }
  } else {
    Blk A, Bb;
    fetch(A);
    for (int i = 0;; i += 2) {
      if (i + 1 >= nblk_run) { reduce(A, true); break; }
      fetch(Bb);
      reduce(A, false);
      if (i + 2 >= nblk_run) { reduce(Bb, true); break; }
      fetch(A);
      reduce(Bb, false);
    }
  }
}

}  // namespace parrot
