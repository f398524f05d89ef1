// Block-diffusion decoding over a KV cache for gfx950: the KV-cache reading
// of DiRL Section 2.1 used in rollouts.  While block k is denoised, its S noisy
// queries attend to the clean tokens of the blocks before it (the cache) and
// to each other in both directions (Eq. 2); nothing else exists yet, so there
// is no mask beyond the lengths.  Every cached K/V row is read once per item
// and serves all of the item's query rows: the work is bound by HBM bandwidth,
// not by the MFMAs.
//
// Work items are (sequence b, KV head, group of the G*S query rows); an item's
// keys are its cache_lens[b] cached rows followed by the block's S rows, cut
// into KT-key tiles (cache tiles, then block tiles; none straddles the two
// arrays).  A team of TW waves, one per 32 query rows, works on an item.  Lay
// the tiles of all items end to end, in item order: T tiles in all.  Team gw of
// the n teams that take part takes the contiguous run [gw*T/n, (gw+1)*T/n),
// whatever the lengths, so every team streams the same number of bytes and a
// long cache is spread over many teams while short ones share one.  The
// lengths live on the device: every workgroup scans them once to find where
// its teams start.  Short calls use fewer teams (dec_runs).
//
// A wave keeps an online-softmax state for the item it is in and flushes it
// when the item or the run ends: an item that lies wholly inside one run is
// written out (O, LSE) at once; otherwise each run leaves its unnormalised O,
// max and sum in a partial slot, and dec_combine_kernel merges the runs of the
// item.  The slot of (gw, item) starts at row gw * rows-per-group + (first row
// of the item's group, all items' rows laid end to end), so slots never
// overlap: two runs (gw, item) and (gw', item') with gw < gw' and item > item'
// cannot both hold tiles, since both the runs and the items are contiguous and
// in the same order.
//
// Teams never wait for each other.  Tiles go straight from HBM to an LDS ring
// of NST stages per team, NST - 1 tiles ahead.
//   TW = 1 (up to 32 query rows per KV head): four teams per workgroup, each
//     wave waits only for its own copies.
//   TW = 2, 4 (up to 64 rows, more): a workgroup is one team, whose waves share
//     each tile, so a KV row is fetched once for up to 128 query rows; one
//     barrier per tile.  24 sequences of 512..8192 tokens, 32 query and 8 KV
//     heads of 128, S = 32 (128 rows per KV head, 370 MB): 91 us; with one wave
//     per 32 rows, which fetched the cache four times, 203 us.  (At 93 us, with
//     tiles of 32 keys 104; with eight waves, half the keys of a tile each, 95.)
// Per tile: S^T = K Q^T (a lane owns a query column, as in the forward pass),
// P = exp2(c S - m) against a lazily moved reference max, O^T += V^T P^T with
// V^T read through the transposing LDS read.
#include "device.hpp"
#include "kernels.hpp"

namespace bd {
namespace {

// The runs that hold an item: first and last, or last = -1 where the decode
// kernel wrote the item directly.
struct alignas(16) DecRuns {
  int first, last;
};

struct DecParams {
  const bf16* Q;   // [B][Hq][S][D]
  const bf16* Kc;  // [B][Hkv][C][D]
  const bf16* Vc;
  const bf16* Kn;  // [B][Hkv][S][D]
  const bf16* Vn;
  const int* cache_lens;  // [B], device
  bf16* O;                // [B][Hq][S][D]
  float* LSE;             // [B][Hq][S]
  DecRuns* desc;          // [item]
  float* part;            // [row][D + 4]: unnormalised O, max (log2 units), sum
  int B, S, Hq, Hkv, G, C;
  int ng;     // row groups per (sequence, KV head)
  int grows;  // query rows of a group (a multiple of 32, at most 32 * TW)
  int hrows;  // partial rows of a (sequence, KV head): its G*S rows rounded up to 32
  int runs;   // teams of the grid
  float c;    // scale * log2(e)
};

// Cache length of sequence b, clamped to [0, C].  `lens` is p.cache_lens
// passed as a restrict kernel argument: the compiler may then read it through
// the scalar cache where the index is uniform.
__device__ inline int dec_len(const DecParams& p, const int* __restrict__ lens, int b) {
  return imin(imax(lens[b], 0), p.C);
}
// Key tiles of an item of a sequence with cache length len.
template <int KT>
__device__ inline int dec_tiles(const DecParams& p, int len) {
  return cdiv(len, KT) + cdiv(p.S, KT);
}
// Teams that take part in a call of T tiles on a grid of `runs` teams: at
// least about DEC_MIN_RUN tiles for each team of several waves, so that a short
// call is not cut into single tiles with as many partial results of its many
// rows to merge (30 sequences of 30 to 60 tokens, S = 32: 15.7 us, single tiles
// 23.0), and no run is empty (T >= 1).  One wave takes single tiles: the same
// time within 2% on one sequence of 1500 tokens, and the nearest to float64,
// since the largest P of a run is 1 exactly (relative error 2.28e-3, with two
// tiles a run 2.32e-3).
template <int TW>
__device__ inline int dec_runs(int runs, int T) {
  constexpr int DEC_MIN_RUN = TW == 1 ? 1 : 2;
  return imin(runs, cdiv(T, DEC_MIN_RUN));
}
// Keys and values of more than 288 MiB, beyond the 256 MiB of the last-level
// cache, are loaded nontemporal: nothing of them survives to the next call, and
// without their lines in L2 and the last-level cache the same bytes come faster
// (822 MB: 150 -> 132 us, 6.2 TB/s).  Smaller ones may still be there from the
// last call, as when a block is denoised step by step.  The line lies where both
// are the same (64 sequences, S = 4, default and nontemporal: 264 MiB 49.9 and
// 50.8 us, 288 MiB 52.4 and 53.9, 296 MiB 56.1 and 56.0, 312 MiB 59.9 and 58.1,
// 336 MiB 68.8 and 61.1).  It holds for rows that a call reads more than once as
// well, by the teams of a KV head's row groups: they run at about the same time
// (256 query rows per KV head: 271 MiB 125 and 131 us, 337 MiB 157 and 156, 412
// MiB 189 and 186, 768 MiB 334 and 324; 512 rows, 375 MiB, the other way round:
// 312 and 316).
constexpr size_t DEC_STREAM_BYTES = (size_t)288 << 20;
// First tile of run gw <= n (the runs cut T tiles into n near-equal pieces).
// RUNS, the teams of the grid, is a power of two, and T <= 2 n where fewer take
// part: no 64-bit division (three of them took 1 us of a call).
template <int RUNS>
__device__ inline int dec_run_start(int gw, int n, int T) {
  return n == RUNS ? (int)(((long long)gw * T) / RUNS) : (int)((unsigned)(gw * T) / (unsigned)n);
}
// First row of the partial slot of run gw for row group g of (sequence, KV head) bh.
__device__ inline size_t dec_slot_row(const DecParams& p, int gw, size_t bh, int g) {
  return (size_t)(gw + g) * p.grows + bh * p.hrows;
}

// Position of a tile: sequence b (cache length len, nt tiles per item), item
// r of the sequence (KV head r / ng, row group r % ng), tile j of the item.
struct DecPos {
  int b, len, nt, r, j;
};

template <int D, int TW, int KT, int NST>
struct DecSmem {
  static constexpr int TEAMS = TW == 1 ? 4 : 1;      // teams per workgroup
  static constexpr int NW = TW * TEAMS;              // waves per workgroup
  static constexpr uint32_t TILE = KT * D * 2;       // bytes of one swizzled K or V tile
  alignas(256) char buf[TEAMS][NST * 2 * TILE];      // per team: a ring of K and V tiles
  int wsum[NW];                                      // prologue: per-wave sums of the scan
  int start_b[TEAMS], start_off[TEAMS];              // where each team's run starts
};

// The reference maximum of a row moves only when the row's scores exceed it
// by more than this (log2 units): P stays below 2^8, well inside bf16 and the
// float32 sums, and most tiles skip the rescale.
constexpr float DEC_SLACK = 8.0f;

template <int D, int TW, int KT, int NST>
__global__ __launch_bounds__(TW == 1 ? 256 : 64 * TW, 1) void dec_kernel(DecParams p, const int* __restrict__ lens) {
  constexpr int DS = D / 16, DB = D / 32, PST = D + 4, KB = KT / 32;
  using Smem = DecSmem<D, TW, KT, NST>;
  constexpr int TEAMS = Smem::TEAMS, NW = Smem::NW, NT = 64 * NW;
  __shared__ Smem sm;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g2 = lane >> 5;
  const int tm = TW == 1 ? w : 0, tw = TW == 1 ? 0 : w;  // team of the workgroup, wave of the team
  const int ng = TW < 4 ? 1 : p.ng;                      // (decode_groups: smaller teams hold all rows of a KV head)
  const int I = p.Hkv * ng;                              // items per sequence

  // ---- prologue: T, and the position of each team's first tile ----
  // thread t sums the tiles per item of sequences [t*cpt, (t+1)*cpt)
  const int cpt = cdiv(p.B, NT);
  const int c0 = imin(p.B, tid * cpt), c1 = imin(p.B, c0 + cpt);
  int csum = 0;
#pragma unroll 4
  for (int b = c0; b < c1; ++b) csum += dec_tiles<KT>(p, dec_len(p, lens, b));
  int incl = csum;  // inclusive scan over the wave
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(incl, o, 64);
    if (lane >= o) incl += u;
  }
  if (lane == 63) sm.wsum[w] = incl;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int v = 0; v < NW; ++v) {
    const int s = sm.wsum[v];
    before += v < w ? s : 0;
    total += s;
  }
  const int excl = before + incl - csum;  // tiles per item of the sequences before c0
  total = __builtin_amdgcn_readfirstlane(total);  // (so that all that follows from it is scalar)
  const int T = total * I;                // checked on the host to fit in 31 bits
  constexpr int RUNS = DEC_WAVES / TW;    // teams of the grid
  const int n = dec_runs<TW>(RUNS, T);
  const bool stream = total * p.Hkv > (int)(DEC_STREAM_BYTES / (2 * Smem::TILE));
  // Run of a workgroup's team v.  Consecutive runs share a workgroup (64
  // sequences of up to 1024 tokens: 28.4 us, 28.8 spread over the workgroups;
  // 32 sequences of 2200, S = 8: 56.0, 57.4), but where fewer teams than the
  // grid holds take part they are spread over the CUs.
  auto run_of = [&](int v) { return n == RUNS ? (int)blockIdx.x * TEAMS + v : v * (int)gridDim.x + (int)blockIdx.x; };
  // the thread whose sequences hold a team's first tile records where it lies
#pragma unroll
  for (int v = 0; v < TEAMS; ++v) {
    const int x0 = dec_run_start<RUNS>(run_of(v), n, T);
    if (csum > 0 && excl * I <= x0 && x0 < (excl + csum) * I) {
      int pb = excl;
      for (int b = c0; b < c1; ++b) {
        const int nt = dec_tiles<KT>(p, dec_len(p, lens, b));
        if (x0 < (pb + nt) * I) {
          sm.start_b[v] = b;
          sm.start_off[v] = x0 - pb * I;
          break;
        }
        pb += nt;
      }
    }
  }
  __syncthreads();

  // ---- this team's run ----
  const int gw = run_of(tm);
  if (gw >= n) return;
  const int x0 = dec_run_start<RUNS>(gw, n, T), x1 = dec_run_start<RUNS>(gw + 1, n, T);
  DecPos pc;
  pc.b = __builtin_amdgcn_readfirstlane(sm.start_b[tm]);
  const int off = __builtin_amdgcn_readfirstlane(sm.start_off[tm]);
  pc.len = __builtin_amdgcn_readfirstlane(dec_len(p, lens, pc.b));
  pc.nt = dec_tiles<KT>(p, pc.len);
  pc.r = off / pc.nt;
  pc.j = off - pc.r * pc.nt;
  const int S = p.S;

  auto advance = [&](DecPos q) __attribute__((always_inline)) {
    if (++q.j == q.nt) {
      q.j = 0;
      if (++q.r == I) {
        q.r = 0;
        if (++q.b < p.B) {
          q.len = __builtin_amdgcn_readfirstlane(dec_len(p, lens, q.b));
          q.nt = dec_tiles<KT>(p, q.len);
        }
      }
    }
    return q;
  };
  // The kernel's arguments, read again.  Those needed once per item do not fit
  // the scalar registers beside what the tile loop itself keeps there: held over
  // the loop they went to vector lanes and a private segment.  (A team of four
  // has no room for those of load_q either; one wave is 2% slower with them
  // read again in front of each item: 8 sequences of up to 4096, S = 16, 23.8 us
  // and 24.4.)
  auto arguments = [&]() __attribute__((always_inline)) -> DecParams {
    auto* a = (const __attribute__((address_space(4))) DecParams*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    return *(const DecParams*)a;
  };
  // this lane's query row of item (b, r): row g*grows + 32*tw + l32 of the G*S
  // rows of KV head r / ng (those rows are consecutive in Q, O and LSE).  A
  // lane past the last row takes the last row instead: its score column is
  // computed like the others (columns never mix) and never stored.
  auto query_row = [&](const DecParams& p, DecPos q, bool& valid) __attribute__((always_inline)) {
    const int hkv = q.r / ng, g = q.r - hkv * ng, rl = 32 * tw + l32, R = g * p.grows + rl;
    valid = R < p.G * S && (TW == 1 || rl < p.grows);
    return ((size_t)q.b * p.Hq + (size_t)hkv * p.G) * S + (R < p.G * S ? R : p.G * S - 1);
  };
  struct QRows {
    bf16x8 v[DS];
  };
  auto load_q = [&](DecPos q) __attribute__((always_inline)) {
    const DecParams a = TW == 4 ? arguments() : p;
    bool valid;
    const size_t row = query_row(a, q, valid);
    QRows r;
#pragma unroll
    for (int s = 0; s < DS; ++s) r.v[s] = *reinterpret_cast<const bf16x8*>(a.Q + row * D + 16 * s + 8 * g2);
    return r;
  };

  const TileCopy<D, KT, 64 * TW> copy(TW == 1 ? lane : tid);  // the team copies a whole tile
  constexpr int NI = decltype(copy)::NI;
  // copy K and V of the tile at q to dst, dst + TILE
  auto issue = [&](DecPos q, char* dst, auto streamed) __attribute__((always_inline)) {
    const size_t grp = (size_t)q.b * p.Hkv + q.r / ng;
    const int ntc = cdiv(q.len, KT);
    const bool cached = q.j < ntc;
    const int r0 = (cached ? q.j : q.j - ntc) * KT;
    const int left = (cached ? q.len : S) - r0;
    const size_t off2 = (cached ? grp * p.C : grp * S) * D + (size_t)r0 * D;
    const bf16 *k = (cached ? p.Kc : p.Kn) + off2, *v = (cached ? p.Vc : p.Vn) + off2;
    constexpr int POLICY = decltype(streamed)::value ? COPY_STREAM : 0;
    copy.template issue_rows<POLICY>(k, left, dst);
    copy.template issue_rows<POLICY>(v, left, dst + Smem::TILE);
  };

  // The whole run, with or without the streaming hint on its copies.  (Twice in
  // the code: a branch around the copies inside a step costs the teams 4%.  All
  // state is the run's own: kept outside, that of the second copy would be held
  // in registers through the first one's loop.)
  auto run = [&](auto streamed) __attribute__((always_inline)) {
    const LdsOperands<D> ops(lane);
    QRows qreg, qnext;
    f32x16 oacc[DB];
    float m, lsum;
    auto reset = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[db][e] = 0.f;
      m = -INFINITY;
      lsum = 0.f;
    };
    reset();
    char* const ring = sm.buf[tm];
    // Query rows first: behind the copies, their latency came on top of the
    // tiles' in front of the first product.
    qreg = load_q(pc);
    // the first NST - 1 tiles (those this run has); pa: the next tile to copy
    DecPos pa = pc;
    issue(pa, ring, streamed);
    pa = advance(pa);
#pragma unroll
    for (int u = 1; u < NST - 1; ++u)
      if (x0 + u < x1) {
        issue(pa, ring + u * 2 * Smem::TILE, streamed);
        pa = advance(pa);
      }
    // Teams: the query rows have landed once all but the newest tile have; one
    // tile at least follows them on every path, so the compiler sees it too (step).
    if (TW > 1) wait_global_loads_but<2 * NI>();

    // Write out the state of the current item's segment, which ends at tile pc.j
    // (tile x of all).
    auto flush = [&](int x) __attribute__((always_inline)) {
      const DecParams p = arguments();
      const int item = pc.b * I + pc.r;
      const int item_start = x - pc.j;  // flat index of the item's first tile
      const bool ends = pc.j == pc.nt - 1;
      bool valid;
      const size_t qrow = query_row(p, pc, valid);
      const float Lrow = halves_sum(lsum);
      if (item_start >= x0 && ends) {
        if (valid) {
          const float inv = 1.f / Lrow;
#pragma unroll
          for (int db = 0; db < DB; ++db) {
            bf16* op = p.O + qrow * D + 32 * db + 4 * g2;
#pragma unroll
            for (int i = 0; i < 4; ++i)
              st_bf16x4(op + 8 * i, oacc[db][4 * i] * inv, oacc[db][4 * i + 1] * inv, oacc[db][4 * i + 2] * inv,
                        oacc[db][4 * i + 3] * inv);
          }
          if (g2 == 0) p.LSE[qrow] = (m + __log2f(Lrow)) * LN2;
        }
        if (lane == 0 && tw == 0) p.desc[item] = DecRuns{0, -1};
        return;
      }
      if (valid) {
        const int hkv = pc.r / ng;
        float* pr = p.part + (dec_slot_row(p, gw, (size_t)pc.b * p.Hkv + hkv, pc.r - hkv * ng) + 32 * tw + l32) * PST;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const f32x4 v = {oacc[db][4 * i], oacc[db][4 * i + 1], oacc[db][4 * i + 2], oacc[db][4 * i + 3]};
            *reinterpret_cast<f32x4*>(pr + 32 * db + 8 * i + 4 * g2) = v;
          }
        if (g2 == 0) *reinterpret_cast<f32x4*>(pr + D) = f32x4{m, Lrow, 0.f, 0.f};
      }
      if (ends && lane == 0 && tw == 0) {
        // the runs holding this item: from the one holding its first tile to this one
        const int first = (int)((((long long)item_start + 1) * n - 1) / T);
        p.desc[item] = DecRuns{first, gw};
      }
    };

    // One tile: `cur` holds the tile at pc; the copy of the tile NST - 1 ahead
    // (at pa, if this run has one) goes to `nxt`, whose last readers are done.
    // The restrict qualifiers tell the compiler that the copy in flight does not
    // touch `cur`, so its reads need not wait for it.
    auto step = [&](const char* __restrict__ cur, char* __restrict__ nxt, DecPos pn, bool more, bool copies,
                    bool new_item) __attribute__((always_inline)) {
      compute_fence();  // the reads of the buffer about to be refilled are done
      if constexpr (TW == 1) {
        // Query rows of the next item (the tile at pn) are loaded a tile ahead,
        // after the wait for the current tile: copies and query loads complete in
        // issue order.  (The query-row copy sits in both branches so that the
        // compiler's own wait for it counts the copy just issued on the first one.)
        if (copies) {
          issue(pa, nxt, streamed);
          wait_global_loads_but<(NST - 1) * 2 * NI>();  // the tile at pc has landed (this wave's own copy)
          if (new_item) qreg = qnext;
          if (pn.j == 0) qnext = load_q(pn);
        } else {
          wait_global_loads();
          if (new_item) qreg = qnext;
        }
      } else {
        // The next item's query rows are loaded a tile ahead here as well, into
        // registers that only the branch that takes them over reads, behind its
        // own wait: were they still in flight at the end of it, the compiler would
        // wait for them, and so for every copy in flight, in front of each tile's
        // first product (121 instead of 95 us for the call above).
        if (new_item) {
          wait_global_loads();
          qreg = qnext;
          compute_fence();  // (keeps this wait from being merged with those below)
        } else if (copies) {
          wait_global_loads_but<(NST - 2) * 2 * NI>();  // this wave's part of the tile at pc has landed
        } else {
          wait_global_loads();
        }
        barrier_lds_only();  // ... every wave's; and all are done with `nxt`
        if (more && pn.j == 0) qnext = load_q(pn);
        if (copies) issue(pa, nxt, streamed);
      }
      const int ntc = cdiv(pc.len, KT);
      const int nvalid = pc.j < ntc ? pc.len - pc.j * KT : S - (pc.j - ntc) * KT;  // keys that exist

      // S^T[key][query] = sum_d K[key][d] Q[query][d]
      f32x16 sacc[KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) sacc[kb][e] = 0.f;
#pragma unroll
      for (int s = 0; s < DS; ++s)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) sacc[kb] = mfma32(lds_rows<D>(cur, ops.row_rel, s, kb), qreg.v[s], sacc[kb]);
      pipeline_lds_reads<DS * KB, 4, 1>();  // operand reads four MFMAs ahead
      if (nvalid < KT) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int i4 = 0; i4 < 4; ++i4)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
              if (32 * kb + 8 * i4 + 4 * g2 + jj >= nvalid) sacc[kb][4 * i4 + jj] = -INFINITY;
      }
      // (row maximum and row sum as balanced trees: no serial chains)
      float m3[KB * 8];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int e = 0; e < 16; e += 2) m3[kb * 8 + e / 2] = fmaxf(sacc[kb][e], sacc[kb][e + 1]);
      const float mx = halves_max(tree_max<KB * 8>(m3)) * p.c;
      const bool grow = mx > m + DEC_SLACK;
      if (__any(grow)) {
        const float alpha = grow ? fast_exp2(m - mx) : 1.f;
        m = grow ? mx : m;
        lsum *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
      }
      bf16x8 pb[2 * KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
        for (int e = 0; e < 16; ++e) sacc[kb][e] = fast_exp2(sacc[kb][e] * p.c - m);
        pb[2 * kb] = pack8(sacc[kb], 0);
        pb[2 * kb + 1] = pack8(sacc[kb], 8);
      }
      lsum += tree_sum<KB>(sacc);
      // O^T[d][query] += sum_key V^T[d][key] P^T[key][query]
#pragma unroll
      for (int c = 0; c < 2 * KB; ++c)
#pragma unroll
        for (int db = 0; db < DB; ++db)
          oacc[db] = mfma32(lds_tr<D>(cur + Smem::TILE, ops.tr_rel0, ops.tr_rel1, c, db), pb[c], oacc[db]);
      // (one wave holds two items' query rows: with reads four MFMAs ahead it
      // runs out of registers and the compiler drops the order altogether)
      pipeline_lds_reads<2 * KB * DB, (TW == 1 ? 3 : 4), 2>();
    };

    uint32_t bcur = 0;                           // ring offset of the tile at pc
    uint32_t bnxt = (NST - 1) * 2 * Smem::TILE;  // ring offset the copy NST - 1 ahead goes to
    for (int x = x0; x < x1; ++x) {
      const DecPos pn = advance(pc);
      const bool more = x + 1 < x1, copies = x + NST - 1 < x1;
      step(ring + bcur, ring + bnxt, pn, more, copies, x > x0 && pc.j == 0);
      if (copies) pa = advance(pa);
      bnxt = bcur;
      bcur = bcur == (NST - 1) * 2 * Smem::TILE ? 0u : bcur + 2 * Smem::TILE;
      if (!more || pn.j == 0) {
        flush(x);
        if (more) reset();  // the next tile starts the next item
      }
      pc = pn;
    }
  };
  if (stream) run(Flag<true>());
  else run(Flag<false>());
}

// Merge the runs of each query row of an item held by several teams:
// O = sum_r 2^(m_r - M) O_r / sum_r 2^(m_r - M) l_r with M = max_r m_r, over
// the runs first..last, merged in one pass (the running maximum moves as runs
// are added, so every run's loads are independent of the others' results).
// One thread per (query row, 4 features, part of the runs): P threads take
// every P-th run each and meet in LDS, in part order.  Rows are those of Q, so
// no thread is spent on padding rows.  Bound by the latency of its dependent
// loads: where few items share the teams (eight runs or more each), P = 8
// (one sequence of 1500 tokens, 24 runs per item: 4 us, against 32 us for one
// thread over the 128 runs it had with empty ones); with more items one
// thread takes the few runs of each (64 sequences: 6.2 us either way).
template <int D, int P>
__global__ __launch_bounds__(256) void dec_combine_kernel(DecParams p) {
  constexpr int TPR = D / 4, PST = D + 4, RPW = 256 / (TPR * P);  // rows per workgroup
  static_assert(RPW >= 1, "a workgroup holds whole rows");
  __shared__ f32x4 so[P > 1 ? 256 : 1];
  __shared__ float2 sml[P > 1 ? 256 : 1];
  const int tid = threadIdx.x;
  const int q4 = tid % TPR, part = (tid / TPR) % P;
  const size_t qrow = (size_t)blockIdx.x * RPW + tid / (TPR * P);  // row of Q: ((b * Hq + h) * S + s)
  const int GS = p.G * p.S;
  DecRuns d = {0, -1};
  float M = -INFINITY, Lr = 0.f;
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  if (qrow < (size_t)p.B * p.Hkv * GS) {
    const int R = (int)(qrow % GS);
    const size_t bh = qrow / GS;  // b * Hkv + hkv
    const int g = R / p.grows, r = R - g * p.grows;
    d = p.desc[bh * p.ng + g];  // (last run -1: written by the decode kernel itself)
#pragma unroll 4
    for (int gw = d.first + part; gw <= d.last; gw += P) {
      const float* ps = p.part + (dec_slot_row(p, gw, bh, g) + r) * PST;
      const f32x4 ml = *reinterpret_cast<const f32x4*>(ps + D);
      const f32x4 v = *reinterpret_cast<const f32x4*>(ps + 4 * q4);
      const float Mn = fmaxf(M, ml[0]);
      const float a = fast_exp2(M - Mn), c = fast_exp2(ml[0] - Mn);  // a = 0 for the first run (M = -inf)
      Lr = Lr * a + ml[1] * c;
      o = o * a + v * c;
      M = Mn;
    }
  }
  if constexpr (P > 1) {
    so[tid] = o;
    sml[tid] = float2{M, Lr};
    __syncthreads();
    if (part != 0 || d.last < 0) return;
    // (part 0 holds at least one run, so M is finite)
#pragma unroll
    for (int u = 1; u < P; ++u) {
      const float2 ml = sml[tid + u * TPR];
      const f32x4 v = so[tid + u * TPR];
      const float Mn = fmaxf(M, ml.x);
      const float a = fast_exp2(M - Mn), c = fast_exp2(ml.x - Mn);  // c = 0 for a part without runs
      Lr = Lr * a + ml.y * c;
      o = o * a + v * c;
      M = Mn;
    }
  } else if (d.last < 0) {
    return;
  }
  const float inv = 1.f / Lr;
  st_bf16x4(p.O + qrow * D + 4 * q4, o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
  if (q4 == 0) p.LSE[qrow] = (M + __log2f(Lr)) * LN2;
}

template <int D, int TW, int KT, int NST>
void launch_dec_kernel(const DecParams& p, hipStream_t st) {
  using Smem = DecSmem<D, TW, KT, NST>;
  hipLaunchKernelGGL((dec_kernel<D, TW, KT, NST>), dim3(p.runs / Smem::TEAMS), dim3(64 * Smem::NW), 0, st, p,
                     p.cache_lens);
}

template <int D>
hipError_t launch_decode_d(const DecodeShape& s, const void* Q, const void* Kc, const void* Vc, const void* Kn,
                           const void* Vn, const int* cache_lens, void* O, float* LSE, void* ws, hipStream_t st) {
  DecParams p;
  p.Q = static_cast<const bf16*>(Q);
  p.Kc = static_cast<const bf16*>(Kc);
  p.Vc = static_cast<const bf16*>(Vc);
  p.Kn = static_cast<const bf16*>(Kn);
  p.Vn = static_cast<const bf16*>(Vn);
  p.cache_lens = cache_lens;
  p.O = static_cast<bf16*>(O);
  p.LSE = LSE;
  p.desc = static_cast<DecRuns*>(ws);
  p.part = reinterpret_cast<float*>(static_cast<char*>(ws) + decode_desc_bytes(s));
  p.B = s.B;
  p.S = s.S;
  p.Hq = s.Hq;
  p.Hkv = s.Hkv;
  p.G = s.Hq / s.Hkv;
  p.C = s.C;
  p.c = s.scale * LOG2E;
  // Row groups: a team of 1, 2 or 4 waves (32 rows each) per group.
  const DecodeGroups g = decode_groups(s);
  p.ng = g.ng;
  p.grows = g.rows;
  p.hrows = DEC_QT * decode_query_tiles(s);
  p.runs = g.runs;
  // (Teams of two take 64 keys a tile at D = 64, half as many barriers: 40
  // sequences of 170 to 398, 64 rows per KV head, 20.2 -> 18.5 us, 19.8 with one
  // wave per 32 rows.  At D = 128 the ring would hold two such tiles.)
  if (g.waves == 1) launch_dec_kernel<D, 1, 32, 2>(p, st);
  else if (g.waves == 2) launch_dec_kernel<D, 2, (D == 64 ? 64 : 32), 4>(p, st);
  else launch_dec_kernel<D, 4, 64, 512 / D>(p, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t rows = (size_t)s.B * s.Hq * s.S, items = (size_t)s.B * s.Hkv * g.ng;
  if (items * 8 <= (size_t)g.runs) {
    constexpr int P = 8, RPW = 256 / (D / 4 * P);
    hipLaunchKernelGGL((dec_combine_kernel<D, P>), dim3((unsigned)((rows + RPW - 1) / RPW)), dim3(256), 0, st, p);
  } else {
    constexpr int RPW = 256 / (D / 4);
    hipLaunchKernelGGL((dec_combine_kernel<D, 1>), dim3((unsigned)((rows + RPW - 1) / RPW)), dim3(256), 0, st, p);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode(const DecodeShape& s, const void* Q, const void* Kc, const void* Vc, const void* Kn,
                         const void* Vn, const int* cache_lens, void* O, float* LSE, void* ws, hipStream_t st) {
  if (s.D == 128) return launch_decode_d<128>(s, Q, Kc, Vc, Kn, Vn, cache_lens, O, LSE, ws, st);
  return launch_decode_d<64>(s, Q, Kc, Vc, Kn, Vn, cache_lens, O, LSE, ws, st);
}

}  // namespace bd
