// Tile binning: the per-tile lists of (tile, Gaussian) intersections, each
// ordered front to back by (float32 camera depth, index).
//
// The lists are built as a counting sort on the tile followed by a sort of
// every list on its own:
//  - each visible Gaussian is counted into the counter of every tile its
//    rectangle covers, so the list lengths are known;
//  - one workgroup scans the lengths into the tile ranges (and orders the
//    tiles longest list first, the order the blend kernels start them in);
//  - every visible Gaussian takes its places in its tiles' ranges through the
//    tiles' cursors, writing the 64-bit key (depth bits << 32 | index). The
//    order inside a range is arbitrary at this point;
//  - one workgroup per tile sorts its range on the key. The keys are unique,
//    so the final lists do not depend on the emission order.
// Every intersection also owns a gradient slot: the Gaussian-major position
// toff[Gaussian] + (its tile's position in the Gaussian's rectangle), from an
// exclusive scan of the tile counts in (view, Gaussian) order. The blend
// backward writes a list entry's gradient into its slot, and the projection
// backward sums a Gaussian's slots, which are contiguous.
#include "internal.h"

namespace asgs {

namespace {

// Inclusive sum over the wave's lanes (mod 2^32): shifts inside the rows of 16
// lanes, then the rows' last lanes broadcast to the rows above.
ASGS_DEV uint32_t wave_incl_scan(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);   // row_shr 1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);   // row_shr 2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);   // row_shr 4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);   // row_shr 8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast 15 -> rows 1, 3
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast 31 -> rows 2, 3
  return x;
}
ASGS_DEV uint32_t last_lane(uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); }

// The block's (view, Gaussian) pair of this thread.
struct ScanBlock {
  int view;
  int64_t j;     // this thread's pair
  bool valid;    // j is a pair of the block
};

ASGS_DEV ScanBlock scan_block(const RenderConst& rc) {
  const int64_t nbx = (rc.n + kScanThreads - 1) / kScanThreads;
  ScanBlock sb;
  sb.view = (int)(blockIdx.x / nbx);
  const int64_t i = (int64_t)(blockIdx.x - sb.view * nbx) * kScanThreads + threadIdx.x;
  sb.valid = i < rc.n;
  sb.j = (int64_t)sb.view * rc.n + i;
  return sb;
}

// ---------------------------------------------------------------------------
// One workgroup: the tile ranges [start, end) from the list lengths, the
// emission cursors (= starts), the totals and the blend order of the tiles
// (per position: tile, start, end), longest list first (a counting sort on the
// length; lengths of 1023 and more share one bucket, and the order within a
// bucket is arbitrary, which changes no result). When the intersections exceed the capacity every range is left
// empty: nothing is blended and the overflow is recorded.
// ---------------------------------------------------------------------------
constexpr int kOrderBins = 1024;
constexpr int kTileScanThreads = 1024;

ASGS_DEV int order_bin(uint32_t c) { return kOrderBins - 1 - (int)(c < kOrderBins - 1 ? c : kOrderBins - 1); }

__global__ void __launch_bounds__(kTileScanThreads) k_tile_scan(RenderConst rc, const ViewDev* __restrict__ views,
                                                               char* ctx, CtxLayout L) {
  constexpr int NW = kTileScanThreads / 64;
  __shared__ uint32_t bins[kOrderBins];
  __shared__ uint32_t scount[ASGS_MAX_VIEWS][kSplitThresholds];  // per view: lists per length band
  __shared__ uint32_t sused[ASGS_MAX_VIEWS], sfrom[ASGS_MAX_VIEWS];  // per view: slots taken, the length they are split from
  __shared__ int32_t sbase[ASGS_MAX_VIEWS + 1];   // first tile of each view
  __shared__ uint32_t svis[ASGS_MAX_VIEWS + 1];   // visible pairs before each view
  __shared__ unsigned long long wtot[NW];
  __shared__ uint32_t wbin[NW], wpb[NW], wpv[NW];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const uint32_t T = (uint32_t)rc.total_tiles;
  uint32_t* tcur = ctx_ptr<uint32_t>(ctx, L.tcur);
  uint2* ranges = ctx_ptr<uint2>(ctx, L.ranges);
  uint4* binfo = ctx_ptr<uint4>(ctx, L.binfo);
  uint4* sinfo = ctx_ptr<uint4>(ctx, L.sinfo);
  CtxHeader* hdr = ctx_ptr<CtxHeader>(ctx, L.hdr);
  // Each wave owns consecutive 64-element chunks of the binning blocks and of
  // the tiles, one element per lane, so that every access is coalesced.
  const uint32_t nbx = (uint32_t)((rc.n + kScanThreads - 1) / kScanThreads);
  const uint32_t nbk = nbx * (uint32_t)rc.n_views;
  const uint32_t perb = ((nbk + 63) / 64 + NW - 1) / NW * 64, pert = ((T + 63) / 64 + NW - 1) / NW * 64;
  const uint32_t b0 = min(nbk, wv * perb), b1 = min(nbk, b0 + perb);
  const uint32_t a0 = min(T, wv * pert), a1 = min(T, a0 + pert);
  // per block: tile-count sum and visible count
  const uint32_t* bs = ctx_ptr<const uint32_t>(ctx, L.bsum);
  const uint32_t* vs = ctx_ptr<const uint32_t>(ctx, L.vsum);
  auto at = [&](const uint32_t* p, uint32_t i, uint32_t end) { return i < end ? p[i] : 0u; };
  bins[t] = 0u;
  for (int q = t; q < rc.n_views * kSplitThresholds; q += kTileScanThreads) (&scount[0][0])[q] = 0u;
  if (t < ASGS_MAX_VIEWS) sused[t] = 0u;
  if (t <= ASGS_MAX_VIEWS) svis[t] = 0u;
  if (t <= rc.n_views) sbase[t] = t < rc.n_views ? views[t].tile_base : (int32_t)T;
  for (int q = t; q < rc.n_views * kSplitPerView; q += kTileScanThreads) sinfo[q] = make_uint4(~0u, 0u, 0u, 0u);
  unsigned long long mine = 0;
  uint32_t pb = 0u, pv = 0u;  // of this wave's blocks
#pragma unroll 4
  for (uint32_t b = b0; b < b1; b += 64) {
    pb += at(bs, b + lane, b1);
    pv += at(vs, b + lane, b1);
  }
  __syncthreads();
  // view of tile i, from the view of an earlier tile
  auto view_from = [&](int v, uint32_t i) {
    while ((int32_t)i >= sbase[v + 1]) ++v;
    return v;
  };
  int v = 0;
  for (uint32_t i0 = a0; i0 < a1; i0 += 64) {
    const uint32_t i = i0 + lane;
    if (i < a1) {
      const uint32_t c = tcur[i];
      mine += c;
      atomicAdd(&bins[order_bin(c)], 1u);
      if (c > (uint32_t)kSplitLen) {
        // band j: kSplitLen + j kSplitStep < c <= kSplitLen + (j + 1) kSplitStep (the last open)
        v = view_from(v, i);
        atomicAdd(&scount[v][min((c - kSplitLen - 1u) / kSplitStep, kSplitThresholds - 1u)], 1u);
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    mine += __shfl_xor(mine, o);
    pb += __shfl_xor(pb, o);
    pv += __shfl_xor(pv, o);
  }
  if (lane == 0) {
    wtot[wv] = mine;
    wpb[wv] = pb;
    wpv[wv] = pv;
  }
  __syncthreads();
  unsigned long long total = 0;
  uint32_t before = 0u, pvt = 0u;
  pb = pv = 0u;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    before += w < wv ? (uint32_t)wtot[w] : 0u;
    total += wtot[w];
    pb += w < wv ? wpb[w] : 0u;
    pv += w < wv ? wpv[w] : 0u;
    pvt += wpv[w];
  }
  // per-block exclusive prefixes for the emission, over all blocks
  {
    uint32_t* bp = ctx_ptr<uint32_t>(ctx, L.bpre);
    uint32_t* vp = ctx_ptr<uint32_t>(ctx, L.vpre);
    uint32_t x = at(bs, b0 + lane, b1), y = at(vs, b0 + lane, b1);
    uint32_t w = nbk ? (b0 + nbx - 1) / nbx : 0u;  // the next view to start
    for (uint32_t b = b0; b < b1; b += 64) {
      const uint32_t xn = at(bs, b + 64 + lane, b1), yn = at(vs, b + 64 + lane, b1);
      const uint32_t ix = wave_incl_scan(x), iy = wave_incl_scan(y);
      if (b + lane < b1) {
        bp[b + lane] = pb + ix - x;
        vp[b + lane] = pv + iy - y;
      }
      for (; w * nbx < min(b1, b + 64); ++w)  // views that start in this chunk
        if (b + lane == w * nbx) svis[w] = pv + iy - y;
      pb += last_lane(ix);
      pv += last_lane(iy);
      x = xn;
      y = yn;
    }
    if (t == 0) svis[rc.n_views] = pvt;
  }
  // places in the blend order: longest class first
  const uint32_t bv = bins[t];
  const uint32_t oincl = wave_incl_scan(bv);
  if (lane == 63) wbin[wv] = oincl;
  __syncthreads();
  uint32_t obefore = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) obefore += w < wv ? wbin[w] : 0u;
  bins[t] = obefore + oincl - bv;
  const bool ovf = total > (unsigned long long)rc.cap;
  if (t == 0) {
    hdr->n_isect = total;
    hdr->n_visible = pvt;
    hdr->overflow = ovf ? 1u : 0u;
  }
  if (t < rc.n_views) {
    ctx_ptr<uint32_t>(ctx, L.vcount)[t] = svis[t + 1] - svis[t];
    // the smallest threshold that few enough lists exceed, from the bands' suffix sums
    uint32_t above = 0u, from = ~0u;
    for (int j = kSplitThresholds - 1; j >= 0 && (above += scount[t][j]) <= (uint32_t)kSplitPerView; --j)
      from = (uint32_t)(kSplitLen + j * kSplitStep);
    sfrom[t] = from;
  }
  __syncthreads();
  uint32_t* bslot = ctx_ptr<uint32_t>(ctx, L.bslot);
  v = 0;
  for (uint32_t i0 = a0; i0 < a1; i0 += 64) {
    const uint32_t i = i0 + lane;
    const uint32_t c = i < a1 ? tcur[i] : 0u;
    const uint32_t incl = wave_incl_scan(c);
    const uint32_t run = before + incl - c;
    before += last_lane(incl);
    if (i < a1) {
      const uint2 r = ovf ? make_uint2(0u, 0u) : make_uint2(run, run + c);
      ranges[i] = r;
      tcur[i] = run;
      binfo[atomicAdd(&bins[order_bin(c)], 1u)] = make_uint4(i, r.x, r.y, 0u);
      // split when longer than the view's threshold (the slot order is arbitrary)
      uint32_t sl = 0u;
      if (!ovf && c > (uint32_t)kSplitLen) {
        v = view_from(v, i);
        if (c > sfrom[v]) {
          const uint32_t slot = (uint32_t)v * kSplitPerView + atomicAdd(&sused[v], 1u);
          sinfo[slot] = make_uint4(i, r.x, r.y, 0u);
          sl = slot + 1u;
        }
      }
      bslot[i] = sl;
    }
  }
}

// ---------------------------------------------------------------------------
// Emission: the exclusive scan of the tile counts in (view, Gaussian) order
// gives every visible Gaussian its first gradient slot; the Gaussian then
// takes one place in the range of every tile of its rectangle. Places are
// reserved per block and tile through the same LDS box as the counting.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kScanThreads) k_dup_emit(RenderConst rc, const ViewDev* __restrict__ views,
                                                           char* ctx, CtxLayout L) {
  __shared__ unsigned long long wred[kScanThreads / 64];
  __shared__ uint32_t wsum[kScanThreads / 64];
  __shared__ uint32_t wvp[kScanThreads / 64], wvc[kScanThreads / 64];
  __shared__ int bred[4];
  __shared__ uint32_t cell[kBoxCells];
  __shared__ RectQueue queue;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const ScanBlock sb = scan_block(rc);
  const ViewDev& V = views[sb.view];
  const uint32_t cnt = sb.valid ? ctx_ptr<const uint32_t>(ctx, L.ntiles)[sb.j] : 0u;
  const short4 r = cnt > 0u ? ctx_ptr<const short4>(ctx, L.rect)[sb.j] : make_short4(1, 0, 1, 0);
  uint32_t* tcur = ctx_ptr<uint32_t>(ctx, L.tcur);
  unsigned long long* ukey = ctx_ptr<unsigned long long>(ctx, L.ukey);
  // first gradient slot: sum of the blocks before this one (the scan's
  // prefix) + the prefix in it
  const unsigned long long pre = ctx_ptr<const uint32_t>(ctx, L.bpre)[blockIdx.x];
  const uint32_t incl = wave_incl_scan(cnt);
  if (lane == 0) wred[wv] = wv == 0 ? pre : 0ull;
  if (lane == 63) wsum[wv] = incl;
  // place in the view's visible list: visible Gaussians of the view's earlier
  // blocks, of the earlier waves, of the earlier lanes
  const int64_t nbx = (rc.n + kScanThreads - 1) / kScanThreads;
  const uint32_t* vpg = ctx_ptr<const uint32_t>(ctx, L.vpre);
  const uint32_t vpre = vpg[blockIdx.x] - vpg[(int64_t)sb.view * nbx];
  const uint64_t vbits = __ballot(cnt > 0u);
  if (lane == 0) {
    wvp[wv] = wv == 0 ? vpre : 0u;
    wvc[wv] = (uint32_t)__popcll(vbits);
  }
  const bool few = V.TX * V.TY <= kBoxCells;  // the grid holds any box
  const bool small = cnt > 0u && (few || cnt <= (uint32_t)kBoxRect);
  const TileBox bx = tile_box(r, small, cnt, bred, cell, queue);  // synchronises: wred, wsum are complete
  unsigned long long off = 0;
  for (int w = 0; w < kScanThreads / 64; ++w) off += wred[w] + (w < wv ? wsum[w] : 0u);
  off += incl - cnt;
  if (sb.valid) ctx_ptr<uint32_t>(ctx, L.toff)[sb.j] = (uint32_t)off;
  if (cnt > 0u) {
    uint32_t vp = __builtin_amdgcn_mbcnt_hi((uint32_t)(vbits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)vbits, 0u));
    for (int w = 0; w < kScanThreads / 64; ++w) vp += wvp[w] + (w < wv ? wvc[w] : 0u);
    ctx_ptr<uint32_t>(ctx, L.vlist)[(int64_t)sb.view * rc.n + vp] = (uint32_t)sb.j;
  }
  // count the block's places per tile, reserve them, then hand them out
  auto cell_of = [&](int tx, int ty) { return (ty - bx.y0) * bx.w + tx - bx.x0; };
  auto via_lds = [&](uint32_t n) { return bx.lds && (few || n <= (uint32_t)kBoxRect); };
  for_tiles(r, cnt, queue, [](int) { return 0; }, [&](int tx, int ty, uint32_t n, int) {
    if (via_lds(n)) atomicAdd(&cell[cell_of(tx, ty)], 1u);
  });
  __syncthreads();
  if (bx.lds)
    for (int c = t; c < bx.area; c += kScanThreads) {
      const uint32_t k = cell[c];
      if (k) {
        const int cy = c / bx.w;
        cell[c] = atomicAdd(&tcur[V.tile_base + (bx.y0 + cy) * V.TX + bx.x0 + c - cy * bx.w], k);
      }
    }
  __syncthreads();
  const uint64_t cap = (uint64_t)rc.cap;
  const uint32_t* dkey = ctx_ptr<const uint32_t>(ctx, L.dkey);
  auto key = [&](int th) {
    const uint32_t j = (uint32_t)(sb.j - t + th);
    return (unsigned long long)dkey[j] << 32 | j;
  };
  for_tiles(r, cnt, queue, key, [&](int tx, int ty, uint32_t n, unsigned long long k) {
    const uint32_t pos = via_lds(n) ? atomicAdd(&cell[cell_of(tx, ty)], 1u)
                                   : atomicAdd(&tcur[V.tile_base + ty * V.TX + tx], 1u);
    if (pos < cap) ukey[pos] = k;
  });
}

// ---------------------------------------------------------------------------
// Per tile: sort the range on the key and write the sorted Gaussian, gradient
// slot and tile key of every list entry. Ranges up to kListSort entries are
// sorted in the workgroup's registers (above 1024 in two runs that are merged in
// LDS); longer ranges are cut into runs of kListSort entries that are sorted the
// same way, which the workgroup then merges pairwise (merge-path split of the output among the threads)
// through a scratch array until one run is left.
// ---------------------------------------------------------------------------
constexpr int kListThreads = 256;
constexpr int kListSort = 2048;
constexpr unsigned long long kKeyMax = ~0ull;  // above every real key (depth bits < 0x7F800000)

// Bitonic sort of 256 K keys in the registers of the workgroup: thread t holds
// keys K t .. K t + K - 1 of the order. Of the steps only three (threads 64 or
// 128 apart) go through LDS and meet at barriers; the others exchange keys
// inside a thread or between the lanes of a wave (data-parallel moves and row
// swaps). Unrolled: as a loop with a branch on the distance a step took 500
// cycles. A list of 169 entries takes 4.5k cycles, 22k with every step
// through LDS; the kernel, which also forms the quarter masks, 9.8 us instead of
// 14.5 at 640x480 (1200 lists of 130 on average), 53 instead of 92 for 8 views of
// 320x240 with 390 on average (7.5 and 42 with masks from the reach box alone).
template <int kCtrl>
ASGS_DEV unsigned long long dpp_move(unsigned long long v) {
  const uint32_t lo = __builtin_amdgcn_update_dpp(0u, (uint32_t)v, kCtrl, 0xF, 0xF, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0u, (uint32_t)(v >> 32), kCtrl, 0xF, 0xF, true);
  return (unsigned long long)hi << 32 | lo;
}
// One step: the thread takes the partner's key where (own > partner) != flip.
template <int K, class Partner>
ASGS_DEV void exchange(unsigned long long (&x)[K], bool flip, Partner partner) {
#pragma unroll
  for (int r = 0; r < K; ++r) {
    const unsigned long long p = partner(x[r]);
    x[r] = (x[r] > p) != flip ? p : x[r];
  }
}
// The same for rows of 16 or halves of 32 lanes: a swap of v with itself gives
// every lane the lower and the upper lane's key.
template <int K, class Swap>
ASGS_DEV void exchange_swap(unsigned long long (&x)[K], bool flip, Swap swap) {
#pragma unroll
  for (int r = 0; r < K; ++r) {
    const auto lo = swap((uint32_t)x[r]), hi = swap((uint32_t)(x[r] >> 32));
    const unsigned long long a = (unsigned long long)hi[0] << 32 | lo[0], b = (unsigned long long)hi[1] << 32 | lo[1];
    x[r] = (a > b) != flip ? b : a;
  }
}
template <int K>
ASGS_DEV void sort_block(unsigned long long (&x)[K], unsigned long long* sk, int t) {
#pragma unroll
  for (int k = 2; k <= 256 * K; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
      const int m = j / K;  // threads apart; 0: inside the thread
      const bool flip = ((t & m) != 0) != ((t & (k / K)) != 0);
      if (m == 0) {
#pragma unroll
        for (int r = 0; r < K; ++r)
          if (!(r & j)) {
            const bool up = ((K * t + r) & k) == 0;
            const unsigned long long a = x[r], b = x[r + j];
            const bool sw = (a > b) == up;
            x[r] = sw ? b : a;
            x[r + j] = sw ? a : b;
          }
      } else if (m == 1) {
        exchange<K>(x, flip, [](unsigned long long v) { return dpp_move<0xB1>(v); });  // quad: 1 0 3 2
      } else if (m == 2) {
        exchange<K>(x, flip, [](unsigned long long v) { return dpp_move<0x4E>(v); });  // quad: 2 3 0 1
      } else if (m == 4) {
        exchange<K>(x, flip, [](unsigned long long v) { return dpp_move<0x1B>(dpp_move<0x141>(v)); });  // 7 - l, 3 - l
      } else if (m == 8) {
        exchange<K>(x, flip, [](unsigned long long v) { return dpp_move<0x128>(v); });  // row rotated by 8
      } else if (m == 16) {
        exchange_swap<K>(x, flip, [](uint32_t v) { return __builtin_amdgcn_permlane16_swap(v, v, false, false); });
      } else if (m == 32) {
        exchange_swap<K>(x, flip, [](uint32_t v) { return __builtin_amdgcn_permlane32_swap(v, v, false, false); });
      } else {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < K; ++r) sk[r * kListThreads + t] = x[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < K; ++r) {
          const unsigned long long p = sk[r * kListThreads + (t ^ m)];
          x[r] = (x[r] > p) != flip ? p : x[r];
        }
      }
    }
  }
}

// Sorts the n keys at a (at most 256 K), leaving them in sk[0, n).
template <int K>
ASGS_DEV void sort_run(const unsigned long long* a, int n, unsigned long long* sk, int t) {
  unsigned long long x[K];
#pragma unroll
  for (int r = 0; r < K; ++r) x[r] = r * kListThreads + t < n ? a[r * kListThreads + t] : kKeyMax;
  sort_block<K>(x, sk, t);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < K; ++r)
    if (K * t + r < n) sk[K * t + r] = x[r];
  __syncthreads();
}

// Sorts the n <= kListSort keys at a into sk[0, n); the caller synchronises
// before sk is used again. Two runs of 1024 are merged, eight outputs per thread
// (their place in the runs by a merge-path search).
ASGS_DEV void sort_keys(const unsigned long long* a, int n, unsigned long long* sk, int t) {
  if (n <= 256) return sort_run<1>(a, n, sk, t);
  if (n <= 512) return sort_run<2>(a, n, sk, t);
  constexpr int kRun = 1024;
  static_assert(kListSort == 2 * kRun && kListSort == 8 * kListThreads, "two runs");
#pragma unroll 1
  for (int c = 0; c < n; c += kRun) sort_run<4>(a + c, min(kRun, n - c), sk + c, t);
  if (n <= kRun) return;
  const unsigned long long* A = sk;
  const unsigned long long* B = sk + kRun;
  const int wb = n - kRun, diag = min(8 * t, n);
  int i0 = max(diag - wb, 0), i1 = min(diag, kRun);
  while (i0 < i1) {
    const int mid = (i0 + i1) >> 1;
    if (A[mid] < B[diag - 1 - mid]) i0 = mid + 1;
    else i1 = mid;
  }
  int i = i0, j = diag - i0;
  unsigned long long x[8], ka = i < kRun ? A[i] : kKeyMax, kb = j < wb ? B[j] : kKeyMax;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const bool fa = ka < kb;
    x[r] = fa ? ka : kb;
    i += fa ? 1 : 0;
    j += fa ? 0 : 1;
    const unsigned long long next = fa ? (i < kRun ? A[i] : kKeyMax) : (j < wb ? B[j] : kKeyMax);
    ka = fa ? next : ka;
    kb = fa ? kb : next;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 8; ++r)
    if (8 * t + r < n) sk[8 * t + r] = x[r];
  __syncthreads();
}

// Which of the tile's four 8x8 quarters (bit w) hold a pixel centre that can
// pass the alpha test power >= ln(alpha_min / o) of an entry: a conservative
// test against the bounding box of the ellipse d^T Q d <= 2 L, Q = [[A, B],
// [B, C]], L = -ln(alpha_min / o), whose half extents are sqrt(2 L C / det Q)
// and sqrt(2 L A / det Q). The box is computed in FP64 from the stored FP32
// conic and widened by a relative 1e-3 + 2e-6 cond(Q) (covering the FP32
// rounding of the per-pixel power, whose error grows with the condition
// number) plus 0.01 px; entries too ill-conditioned for that bound are kept
// everywhere. Entries whose threshold no pixel can reach (o < alpha_min, or
// a NaN threshold) are dropped everywhere. The masks decide where the forward
// cuts a quarter's list in two, and with it the last bits of T.
// Entries whose reach box, which holds that box and was written by the
// projection (two half-precision extents), misses the tile are dropped first.
ASGS_DEV uint32_t quarter_mask(const float4& g0, const float4& g1, int x0, int y0) {
  const float lnthr = g1.z;
  const uint32_t box = __float_as_uint(g1.w);
  const float bx = (float)__builtin_bit_cast(_Float16, (uint16_t)box);
  const float by = (float)__builtin_bit_cast(_Float16, (uint16_t)(box >> 16));
  const float tx0 = (float)x0, ty0 = (float)y0;
  if (!(g0.x + bx >= tx0 && g0.x - bx <= tx0 + (float)(kTile - 1) && g0.y + by >= ty0 &&
        g0.y - by <= ty0 + (float)(kTile - 1)))
    return 0u;
  if (!(lnthr <= 0.f)) return 0u;
  const double a = g0.z, b = g0.w, c = g1.x;
  const double det = a * c - b * b;
  if (!(det > 0.0) || !(a > 0.0) || !(c > 0.0)) return 0xFu;
  const double half_tr = 0.5 * (a + c);
  const double disc = sqrt(0.25 * (a - c) * (a - c) + b * b);
  const double lmax = half_tr + disc;
  const double cond = lmax * lmax / det;  // lmax / lmin
  const double rel = 1e-3 + 2e-6 * cond;
  if (!(rel < 0.25)) return 0xFu;
  const double L2 = -2.0 * (double)lnthr;
  const double hx = sqrt(L2 * c / det) * (1.0 + rel) + 0.01;
  const double hy = sqrt(L2 * a / det) * (1.0 + rel) + 0.01;
  const double u = g0.x, v = g0.y;
  uint32_t m = 0u;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const double sx = x0 + 8 * (w & 1), sy = y0 + 8 * (w >> 1);
    if (u + hx >= sx && u - hx <= sx + 7.0 && v + hy >= sy && v - hy <= sy + 7.0) m |= 1u << w;
  }
  return m;
}

struct ListOut {
  const float* geom;
  uint8_t* pmask;
  const short4* rect;
  const uint32_t* toff;
  uint32_t* pairgid;
  uint32_t* pslot;
  uint32_t* ptile;
  uint32_t tile;
  int tx, ty;

  // Gaussian, gradient slot, tile and quarter mask of list position pos.
  ASGS_DEV void put(uint64_t pos, unsigned long long key) const {
    const uint32_t gid = (uint32_t)key;
    const short4 r = rect[gid];
    const float4* g = reinterpret_cast<const float4*>(geom + (size_t)gid * kGeomStride);
    pairgid[pos] = gid;
    pmask[pos] = (uint8_t)quarter_mask(g[0], g[1], tx * kTile, ty * kTile);
    pslot[pos] = toff[gid] + (uint32_t)((ty - r.z) * (r.y - r.x + 1) + (tx - r.x));
    ptile[pos] = tile;
  }
};

__global__ void __launch_bounds__(kListThreads) k_list_sort(RenderConst rc, const ViewDev* __restrict__ views,
                                                           char* ctx, CtxLayout L) {
  __shared__ unsigned long long sk[kListSort];
  const uint4 bi = ctx_ptr<const uint4>(ctx, L.binfo)[blockIdx.x];
  const uint32_t tile = bi.x;
  const uint2 rg = make_uint2(bi.y, bi.z);
  const uint32_t n = rg.y - rg.x;
  if (n == 0u) return;
  const int t = threadIdx.x;
  ListOut out;
  {
    const ViewDev& V = views[find_view(views, rc.n_views, (int)tile)];
    const int lt = (int)tile - V.tile_base;
    out.ty = lt / V.TX;
    out.tx = lt - out.ty * V.TX;
  }
  out.geom = ctx_ptr<const float>(ctx, L.geom);
  out.pmask = ctx_ptr<uint8_t>(ctx, L.pmask);
  out.rect = ctx_ptr<const short4>(ctx, L.rect);
  out.toff = ctx_ptr<const uint32_t>(ctx, L.toff);
  out.pairgid = ctx_ptr<uint32_t>(ctx, L.pairgid);
  out.pslot = ctx_ptr<uint32_t>(ctx, L.pslot);
  out.ptile = ctx_ptr<uint32_t>(ctx, L.ptile);
  out.tile = tile;
  unsigned long long* a = ctx_ptr<unsigned long long>(ctx, L.ukey) + rg.x;
  if (n <= (uint32_t)kListSort) {
    sort_keys(a, (int)n, sk, t);
    for (uint32_t i = t; i < n; i += kListThreads) out.put(rg.x + i, sk[i]);
    return;
  }
  // sorted runs of kListSort entries, in place
  for (uint32_t c0 = 0; c0 < n; c0 += kListSort) {
    const uint32_t m = min((uint32_t)kListSort, n - c0);
    sort_keys(a + c0, (int)m, sk, t);
    for (uint32_t i = t; i < m; i += kListThreads) a[c0 + i] = sk[i];
    __syncthreads();
  }
  // pairwise merges of runs of width w, a -> b, until one run is left
  unsigned long long* b = ctx_ptr<unsigned long long>(ctx, L.tkey) + rg.x;
  const uint64_t per = ((uint64_t)n + kListThreads - 1) / kListThreads;
  for (uint64_t w = kListSort; w < n; w <<= 1) {
    uint64_t o = min((uint64_t)n, (uint64_t)t * per);
    const uint64_t oend = min((uint64_t)n, o + per);
    while (o < oend) {
      const uint64_t lo = o - o % (2 * w);
      const uint64_t wa = min(w, (uint64_t)n - lo);
      const uint64_t wb = min(w, (uint64_t)n - lo - wa);
      const unsigned long long* A = a + lo;
      const unsigned long long* B = A + wa;
      const uint64_t diag = o - lo;
      // entries of A among the first diag outputs of this merge
      uint64_t i0 = diag > wb ? diag - wb : 0, i1 = min(diag, wa);
      while (i0 < i1) {
        const uint64_t mid = (i0 + i1) >> 1;
        if (A[mid] < B[diag - 1 - mid]) i0 = mid + 1;
        else i1 = mid;
      }
      uint64_t i = i0, j = diag - i0;
      const uint64_t stop = min(oend, lo + wa + wb);
      unsigned long long ka = i < wa ? A[i] : kKeyMax, kb = j < wb ? B[j] : kKeyMax;
      for (; o < stop; ++o) {
        if (ka < kb) {
          b[o] = ka;
          ++i;
          ka = i < wa ? A[i] : kKeyMax;
        } else {
          b[o] = kb;
          ++j;
          kb = j < wb ? B[j] : kKeyMax;
        }
      }
    }
    __syncthreads();
    unsigned long long* tmp = a;
    a = b;
    b = tmp;
  }
  for (uint32_t i = t; i < n; i += kListThreads) out.put(rg.x + i, a[i]);
}

}  // namespace

void launch_bin(const RenderConst& rc, const CtxLayout& L, char* ctx, hipStream_t s) {
  const unsigned nblk = (unsigned)scan_blocks(rc.n, rc.n_views);
  const ViewDev* views = reinterpret_cast<const ViewDev*>(ctx + L.views);
  hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(kTileScanThreads), 0, s, rc, views, ctx, L);
  if (nblk > 0) hipLaunchKernelGGL(k_dup_emit, dim3(nblk), dim3(kScanThreads), 0, s, rc, views, ctx, L);
}

void launch_tile_sort(const RenderConst& rc, const CtxLayout& L, char* ctx, hipStream_t s) {
  const ViewDev* views = reinterpret_cast<const ViewDev*>(ctx + L.views);
  hipLaunchKernelGGL(k_list_sort, dim3(rc.total_tiles), dim3(kListThreads), 0, s, rc, views, ctx, L);
}

}  // namespace asgs
