// Front-to-back alpha compositing of colour, depth and the low-dimensional
// feature (UP-SLAM Sec. 3.1 Eq. 3, Sec. 3.3 Eq. 10) and its backward.
//
// A wave covers an 8x8 quarter of a 16x16 screen tile, a pixel per lane. It
// visits the entries of the tile's depth-ordered list whose alpha >= alpha_min
// ellipse can reach the quarter (the mask the list sort left with each entry);
// an entry is the same for all lanes, so its record comes through scalar loads,
// one entry ahead, and takes no vector register or LDS. Each pixel skips alpha
// < alpha_min, stops before the transmittance would fall below T_min, and
// accumulates w = alpha * T times (rgb, z, feature). In the forward a workgroup
// is one quarter (two waves, each a half of a round of the list), and leaves as
// soon as its pixels have stopped.
//
// The backward (a workgroup per tile or segment of a long list, a wave per
// quarter) replays each pixel's list back to front from its last composited
// Gaussian, recovering T_k = T_{k+1} / (1 - alpha_k), and sums each entry's
// gradient over the tile's pixels on the matrix cores (see k_blend_bwd); every
// entry's gradient slot is written once, without global atomics. The projection
// backward then sums each Gaussian's slots.
#include "internal.h"

namespace asgs {

namespace {

// Pixel of thread t: wave w covers the 8x8 quarter (w & 1, w >> 1) of the
// tile, lane l the pixel (l & 7, l >> 3) inside it. Square quarters keep the
// per-wave culling below tight.
ASGS_DEV int tile_lx(int t) { return ((t >> 6) & 1) * 8 + (t & 7); }
ASGS_DEV int tile_ly(int t) { return ((t >> 7) & 1) * 8 + ((t >> 3) & 7); }

// Issue priority of a workgroup's waves by its rank in the launch: the blend
// order (longest list first), in the backward behind the places of the split
// lists' segments. The first workgroups of a launch spread over the compute
// units, so the first on each unit gets the highest priority, the next one the
// next level: they are preferred over the shorter ones sharing their SIMDs (the
// order of the results does not change). With four views and more the segments' places,
// used or not, take all levels of the backward.
ASGS_DEV void prioritise(uint32_t rank, int n_cu) {
  const uint32_t band = rank / (uint32_t)(n_cu > 0 ? n_cu : 1);
  if (band == 0u) __builtin_amdgcn_s_setprio(3);
  else if (band == 1u) __builtin_amdgcn_s_setprio(2);
  else if (band == 2u) __builtin_amdgcn_s_setprio(1);
}

ASGS_DEV bool any_lane(bool b) { return __builtin_amdgcn_ballot_w64(b) != 0; }

// A Gaussian's blend record in scalar registers: geometry (u, v, A, B, C, o,
// ln(alpha_min / o)) and channels. The loads go through the constant address
// space, so a wave-uniform index makes them scalar loads.
typedef float f4u __attribute__((ext_vector_type(4), aligned(16)));
typedef float f8u __attribute__((ext_vector_type(8), aligned(16)));
typedef float f16u __attribute__((ext_vector_type(16), aligned(16)));
#define ASGS_CONST_AS __attribute__((address_space(4)))

template <int CS>
struct SRec;
template <>
struct SRec<4> {
  f8u g;
  f4u c;
  ASGS_DEV void load(const float* geom, const float* chan, uint32_t gid) {
    g = *(const ASGS_CONST_AS f8u*)(geom + (size_t)gid * kGeomStride);
    c = *(const ASGS_CONST_AS f4u*)(chan + (size_t)gid * 4);
  }
  ASGS_DEV float ch(int k) const { return c[k]; }
  // The unused last word stays allocated until the record is used: its
  // register, reused earlier, would have to wait for the load in flight.
  ASGS_DEV void keep() const { asm volatile("" ::"s"(g[7])); }
};
template <>
struct SRec<20> {
  f8u g;
  f16u c;
  f4u d;
  ASGS_DEV void load(const float* geom, const float* chan, uint32_t gid) {
    g = *(const ASGS_CONST_AS f8u*)(geom + (size_t)gid * kGeomStride);
    const float* p = chan + (size_t)gid * 20;
    c = *(const ASGS_CONST_AS f16u*)p;
    d = *(const ASGS_CONST_AS f4u*)(p + 16);
  }
  ASGS_DEV float ch(int k) const { return k < 16 ? c[k < 16 ? k : 0] : d[k < 16 ? 0 : k - 16]; }
  ASGS_DEV void keep() const { asm volatile("" ::"s"(g[7])); }
};

constexpr int kSplitMin = 16;     // a round's quarter list shorter than this stays on the front wave

// Forward compositing, one workgroup of two waves per 8x8 quarter of a tile.
// Per round of the list (256 entries, kSeg of a split list), the entries that
// can reach one of the quarter's pixels (the sort's quarter masks) are split in
// list order: the front wave composites the first half onto the running
// state (T, channels, last contributor), the back wave the second half from
// T = 1 at the same time, both with the records in scalar registers (requested
// one entry ahead, their cache lines touched at the start of the round); then
// the front wave appends the back half's result,
//   C <- C + T C_back,  T <- T T_back,
// which equals compositing the two halves in order as long as the
// transmittance cannot have crossed T_min inside the back half
// (T T_back >= T_min, T being monotone). Pixels where it could re-run the
// back half on the front wave with the sequential rule.
//
// The rounds and halves are part of the result: they set the last bits of T,
// and the second moments of the backward carry FP32 rounding that such bits
// redraw (up to 1e-3 of the rms at single elements of the anchors' feature
// gradient). Rounds of 128 and, in small views, four waves per quarter change
// them; they would be faster where lists are long (a 640x480 view through a
// volume 89 us instead of 99, eight 320x240 keyframes 162 instead of 202).
//
// Bound by the vector ALU (about 42 instructions per used entry) and, on few
// tiles, by the longest lists. One 512-thread workgroup per tile with the
// records staged through LDS waited at its barriers two thirds of the time:
// one 640x480 view of 157k intersections 48 us, now 31; 774k intersections 267,
// now 157; eight 320x240 views with 986k 339, now 202; 80 tiles of 50k (no
// features) 71, now 41.
//
// With L1, the output stage also forms the weighted L1 residual of the maps
// against the targets and its gradient (the terms of the L1 loss kernel, in
// the same arithmetic), and each quarter's loss partial.
ASGS_DEV float l1_sgn(float d) { return d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f); }

constexpr int kFwdWaves = 2;
template <int NF, bool L1>
__global__ void __launch_bounds__(64 * kFwdWaves) k_blend_fwd(RenderConst rc, const ViewDev* __restrict__ views,
                                                           char* ctx, CtxLayout L, asgs_images out, BlendL1 l1) {
  constexpr int CS = 4 + NF;
  constexpr int kRound = 256;  // the longest round
  // 32 consecutive workgroups are the four quarters of eight tiles, those of a
  // tile eight apart, so that they share an XCD's L2 (workgroups go to the
  // XCDs round-robin)
  const uint32_t bpos = (blockIdx.x >> 5) * 8u + (blockIdx.x & 7u);
  const int qd = (blockIdx.x >> 3) & 3;
  if (bpos >= (uint32_t)rc.total_tiles) return;
  const uint4 bi = ctx_ptr<const uint4>(ctx, L.binfo)[bpos];  // longest lists first
  const int tile = (int)bi.x;
  const int view = find_view(views, rc.n_views, tile);
  const ViewDev& V = views[view];
  const int lt = tile - V.tile_base;
  const int ty = lt / V.TX, tx = lt - ty * V.TX;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool back = wv > 0;  // back half of the round's list
  const int tq = (qd << 6) | lane;
  const int px = tx * kTile + tile_lx(tq);
  const int py = ty * kTile + tile_ly(tq);
  const bool inside = px < V.W && py < V.H;
  const float pxf = (float)px, pyf = (float)py;
  const uint2 rg = make_uint2(bi.y, bi.z);
  prioritise(bpos, rc.n_cu);
  const uint32_t* pairgid = ctx_ptr<const uint32_t>(ctx, L.pairgid);
  const float* geom = ctx_ptr<const float>(ctx, L.geom);
  const float* chan = ctx_ptr<const float>(ctx, L.chan);
  const uint8_t* pmask = ctx_ptr<const uint8_t>(ctx, L.pmask);
  // lists walked by several backward workgroups: taken kSeg entries at a
  // time, with the pixel's state recorded at every segment boundary
  static_assert(split_floats(CS) == ((kSegMax - 1) * split_first(CS) + split_final(CS)) * kTilePix, "segment layout");
  const uint32_t sl = ctx_ptr<const uint32_t>(ctx, L.bslot)[tile];  // 1 + split-record slot, or 0
  const int nseg = sl ? split_segments(rg.y - rg.x) : 1;
  const uint32_t rstep = nseg > 1 ? (uint32_t)kSeg : (uint32_t)kRound;  // entries per round
  constexpr int SA = split_first(CS), SF = split_final(CS);
  float* sp = ctx_ptr<float>(ctx, L.split) + (size_t)(sl ? sl - 1u : 0u) * split_floats(CS);

  __shared__ uint2 swl[kRound];                     // the quarter's entries of the round (every wave writes the same)
  __shared__ float xch[CS + 2][64];  // back half's state per pixel: T, channels, last
  __shared__ uint64_t qdone;         // front lanes already stopped

  // L1 targets and weight of the pixel, requested now and used in the output stage
  float tv[CS + 1], tw = 1.f;
  if (L1) {
#pragma unroll
    for (int c = 0; c <= CS; ++c) tv[c] = 0.f;
    if (!back && inside) {
      const size_t HW = (size_t)V.W * V.H;
      const size_t pix = (size_t)py * V.W + px;
      const size_t pb = (size_t)V.pix_base;
      if (l1.w) tw = l1.w[pix];
      if (l1.t[0])
        for (int c = 0; c < 3; ++c) tv[c] = l1.t[0][3 * pb + c * HW + pix];
      if (l1.t[1]) tv[3] = l1.t[1][pb + pix];
      if (NF > 0 && l1.t[2]) {
#pragma unroll
        for (int c = 0; c < NF; ++c) tv[4 + c] = l1.t[2][NF * pb + c * HW + pix];
      }
      if (l1.t[3]) tv[CS] = l1.t[3][pb + pix];
    }
  }

  float T = 1.f;
  float acc[CS];
#pragma unroll
  for (int c = 0; c < CS; ++c) acc[c] = 0.f;
  uint32_t last = 0;
  bool done = back || !inside;  // back lanes keep no running state
  const float amax = rc.alpha_max, tmin = rc.T_min;
  // Composite the positions [i0, i1) of this wave's list of the round on the
  // lanes with reach = 0 (others: -inf, below every power); a lane stops
  // (reach = -inf) before T would fall below tstop (T_min, or -1 for the local
  // back half's state).
  constexpr float kNoReach = -__builtin_inff();
  auto run = [&](int i0, int i1, float& reach, float tstop) {
    const uint2* lst = swl;
    // one entry at list position pos; false when every lane has stopped
    auto entry = [&](const SRec<CS>& rec, uint32_t pos) -> bool {
      rec.keep();
      float dx, dy;
      const float power = eval_power(rec.g[0], rec.g[1], rec.g[2], rec.g[3], rec.g[4], pxf, pyf, dx, dy);
      // alpha >= alpha_min  <=>  power >= ln(alpha_min / o) (record slot 6)
      const bool use = power <= reach && power >= rec.g[6];
      if (!any_lane(use)) return true;
      const float alpha = fminf(amax, rec.g[5] * __expf(power));
      const float Tn = T * (1.f - alpha);
      const bool stop = use && Tn < tstop;
      if (use && !stop) {
        const float w = alpha * T;
#pragma unroll
        for (int k = 0; k < CS; ++k) acc[k] = fmaf(w, rec.ch(k), acc[k]);
        T = Tn;
        last = pos;
      }
      if (any_lane(stop)) {
        reach = stop ? kNoReach : reach;
        return any_lane(reach == 0.f);
      }
      return true;
    };
    SRec<CS> ra, rb;
    uint2 ea = lst[i0], eb = lst[min(i0 + 1, i1 - 1)];
    ra.load(geom, chan, (uint32_t)__builtin_amdgcn_readfirstlane((int)ea.x));
    for (int i = i0;;) {
      rb.load(geom, chan, (uint32_t)__builtin_amdgcn_readfirstlane((int)eb.x));
      const uint32_t pa = ea.y;
      ea = lst[min(i + 2, i1 - 1)];
      if (!entry(ra, pa) || ++i >= i1) break;
      ra.load(geom, chan, (uint32_t)__builtin_amdgcn_readfirstlane((int)ea.x));
      const uint32_t pb = eb.y;
      eb = lst[min(i + 2, i1 - 1)];
      if (!entry(rb, pb) || ++i >= i1) break;
    }
  };
  // the round's Gaussian ids and quarter masks, lane l entry 64 k + l
  uint32_t gid[kRound / 64], msk[kRound / 64];
  auto fetch = [&](uint32_t base) {
    const uint32_t end = min(rg.y, base + rstep);
#pragma unroll
    for (int k = 0; k < kRound / 64; ++k) {
      const uint32_t p = base + 64 * k + lane;
      gid[k] = p < end ? pairgid[p] : 0u;
      msk[k] = p < end ? pmask[p] : 0u;
    }
  };
  fetch(rg.x);
  for (uint32_t base = rg.x; base < rg.y; base += rstep) {
    {
      const uint64_t dm = __ballot(done);
      if (!back && lane == 0) qdone = dm;
    }
    __syncthreads();
    const uint64_t dm = qdone;
    if (!~dm) break;
    // the quarter's entries of the round (those that can reach one of its
    // pixels), in list order, compacted into swl (the same list on every wave):
    // the Gaussian and the position in the tile's list plus one
    int n = 0;
#pragma unroll
    for (int k = 0; k < kRound / 64; ++k) {
      const bool mine = (msk[k] >> qd) & 1u;
      const uint64_t bits = __ballot(mine);
      if (mine)
        swl[n + __builtin_amdgcn_mbcnt_hi((uint32_t)(bits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bits, 0u))] =
            make_uint2(gid[k], base - rg.x + 64 * k + lane + 1u);
      n += __builtin_popcountll(bits);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int nf = n < kSplitMin ? n : (n + 1) / 2;  // the front half
    const int p0 = back ? nf : 0, p1 = back ? n : nf;
    // touch the records of this wave's half, and request the next round's ids
    float touch = 0.f;
    for (int i = p0 + lane; i < p1; i += 64) {
      const size_t g = swl[i].x;
      touch += geom[g * kGeomStride] + chan[g * CS] + chan[g * CS + CS - 1];
    }
    fetch(base + rstep);
    if (back) {
      T = 1.f;
#pragma unroll
      for (int c = 0; c < CS; ++c) acc[c] = 0.f;
      last = 0u;
      const bool skip = !inside || ((dm >> lane) & 1u);
      float reach = skip ? kNoReach : 0.f;
      if (p0 < p1) run(p0, p1, reach, -1.f);
      xch[0][lane] = T;
#pragma unroll
      for (int c = 0; c < CS; ++c) xch[1 + c][lane] = acc[c];
      xch[CS + 1][lane] = __uint_as_float(last);
    } else if (n > 0) {
      float reach = done ? kNoReach : 0.f;
      run(0, nf, reach, tmin);
      done = reach != 0.f;
    }
    asm volatile("" ::"v"(touch));  // the touching loads are kept, and waited for here
    __syncthreads();
    if (!back && nf != n) {
      // append the back half
      const float Tb = xch[0][lane];
      const uint32_t lastb = __float_as_uint(xch[CS + 1][lane]);
      const bool fix = !done && T * Tb < tmin;
      if (!done && !fix) {
#pragma unroll
        for (int c = 0; c < CS; ++c) acc[c] = fmaf(T, xch[1 + c][lane], acc[c]);
        T *= Tb;
        if (lastb) last = lastb;
      }
      if (any_lane(fix)) {
        float reach = fix ? 0.f : kNoReach;
        run(nf, n, reach, tmin);
        done = done || (fix && reach != 0.f);
      }
    }
    const int bnd = (int)((base - rg.x) / kSeg) + 1;  // segment boundary after this round
    if (nseg > 1 && !back && bnd < nseg) {
      // state after the first bnd * kSeg entries
      float* rp = sp + ((size_t)(bnd - 1) * kTilePix + tq) * SA;
      float r[SA];
      r[0] = T;
#pragma unroll
      for (int c = 0; c < CS; ++c) r[1 + c] = acc[c];
#pragma unroll
      for (int c = 1 + CS; c < SA; ++c) r[c] = 0.f;
#pragma unroll
      for (int c4 = 0; c4 < SA / 4; ++c4)
        reinterpret_cast<float4*>(rp)[c4] = make_float4(r[4 * c4], r[4 * c4 + 1], r[4 * c4 + 2], r[4 * c4 + 3]);
    }
  }
  if (nseg > 1 && !back) {
    // the final channels (the entries after a boundary add C_final - C_boundary)
    float* rp = sp + (size_t)(kSegMax - 1) * kTilePix * SA + (size_t)tq * SF;
    float r[SF];
#pragma unroll
    for (int c = 0; c < SF; ++c) r[c] = c < CS ? acc[c < CS ? c : 0] : 0.f;
#pragma unroll
    for (int c4 = 0; c4 < SF / 4; ++c4)
      reinterpret_cast<float4*>(rp)[c4] = make_float4(r[4 * c4], r[4 * c4 + 1], r[4 * c4 + 2], r[4 * c4 + 3]);
  }
  if (back) return;
  float lsum = 0.f;  // this pixel's L1 loss terms
  if (inside) {
    const size_t HW = (size_t)V.W * V.H;
    const size_t pix = (size_t)py * V.W + px;
    const size_t pb = (size_t)V.pix_base;
    float map[CS + 1];  // rgb, depth, feature, opacity sum
    map[0] = acc[0] + T * rc.bg[0];
    map[1] = acc[1] + T * rc.bg[1];
    map[2] = acc[2] + T * rc.bg[2];
#pragma unroll
    for (int c = 3; c < CS; ++c) map[c] = acc[c];
    map[CS] = 1.f - T;
#pragma unroll
    for (int c = 0; c < 3; ++c) out.rgb[3 * pb + c * HW + pix] = map[c];
    out.depth[pb + pix] = map[3];
    if (NF > 0) {
#pragma unroll
      for (int c = 0; c < NF; ++c) out.feat[NF * pb + c * HW + pix] = map[4 + c];
    }
    out.alpha[pb + pix] = map[CS];
    ctx_ptr<float>(ctx, L.tfinal)[pb + pix] = T;
    ctx_ptr<uint32_t>(ctx, L.ncontrib)[pb + pix] = last;
    if (L1) {
      const float w = tw;
      // group q: channels [c0, c0 + nc) of the maps, plane base of view v
      auto group = [&](int q, int c0, int nc, size_t vbase) {
        float* g = l1.g[q];
        if (!l1.t[q]) {
          if (g)
            for (int c = 0; c < nc; ++c) g[vbase + c * HW + pix] = 0.f;
          return;
        }
        float l = 0.f;
        for (int c = 0; c < nc; ++c) {
          const float d = map[c0 + c] - tv[c0 + c];
          l += fabsf(d);
          if (g) g[vbase + c * HW + pix] = w * l1_sgn(d) * l1.s[q];
        }
        lsum += w * l * l1.s[q];
      };
      group(0, 0, 3, 3 * pb);
      group(1, 3, 1, pb);
      if (NF > 0) group(2, 4, NF, NF * pb);
      group(3, CS, 1, pb);
    }
  }
  if (L1) {
    for (int o = 32; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o);
    if (lane == 0) ctx_ptr<float>(ctx, L.lpart)[4 * tile + qd] = lsum;
  }
}

// Per view: the fused forward's loss, a fixed-order sum of its tiles' quarter
// partials.
__global__ void __launch_bounds__(256) k_l1_tile_loss(const ViewDev* __restrict__ views, const float* lpart,
                                                      float* loss) {
  __shared__ float red[256 / 64];
  const ViewDev& V = views[blockIdx.x];
  const int nt = V.TX * V.TY;
  float s = 0.f;
  for (int t = threadIdx.x; t < nt; t += blockDim.x) {
    const float* p = lpart + 4 * (size_t)(V.tile_base + t);
    s += (p[0] + p[1]) + (p[2] + p[3]);
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) loss[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

constexpr int kBwdBatch = 8;  // list entries per MFMA tile: rows 0-7 hold w, rows 8-15 dL/dpower

typedef float f4v __attribute__((ext_vector_type(4)));

typedef __bf16 bf8v __attribute__((ext_vector_type(8)));

ASGS_DEV f4v mfma_bf(const bf8v& a, const bf8v& b, f4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Round to nearest even bfloat16 (the hardware conversion of gfx950).
ASGS_DEV uint16_t bf_rne(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
// v = hi + lo with hi = bf16(v) and lo = bf16(v - hi), both rounded to nearest
// even: |v - hi - lo| <= 2^-17 |v| for finite v. With exact bf16 products and
// FP32 accumulation, a b ~ ah bh + ah bl + al bh to ~2^-15 relative.
ASGS_DEV void bf_split(float v, uint16_t& hi, uint16_t& lo) {
  hi = bf_rne(v);
  lo = bf_rne(v - __uint_as_float((uint32_t)hi << 16));
}

// Backward compositing, one workgroup per tile (or per 128-entry segment of
// a split list), one pixel per thread.
//
// Per list entry k and pixel p the gradient contributions are
//   dL/dc_k      += w_kp G_p                 (w = alpha T, G = upstream channel gradients)
//   dL/dpower_kp  = dL/dalpha_kp * alpha_kp  (0 when alpha is clamped)
//   dL/do_k      += dL/dpower_kp / o_k
//   dL/du_k       = -sum_p dpow (A dx + B dy), ...  with dx = u - px, dy = v - py
// so the per-entry sums over the tile's pixels are dot products of two
// per-pixel coefficients (w, dpow) with fixed per-pixel features: the
// channel gradients G_p and the moments (1, lx, ly, lx^2, lx ly, ly^2) of the
// tile-local pixel coordinates, from which the conic and position gradients
// follow in closed form. The list is walked in rounds
// of 32 entries from the back. Each wave takes only the round's entries that
// one of its pixels uses (the quarter test of the forward, then a ballot);
// their records arrive through scalar loads, one entry ahead, so the channel
// dot product takes them as scalar operands and no record passes through LDS.
// The pixels' coefficients of up to 8 such entries go to LDS as the 16 rows
// of one matrix-core tile (8 rows of w, 8 of dL/dpower) and are contracted
// over the wave's 64 pixels (bf16 16x16x32 MFMAs with both operands split
// into hi + lo parts) against the channel gradients and the moments. At the
// end of a round each wave turns its rows' moments into the gradients of
// (u, v, A, B, C, o), and the four waves' rows are summed in a fixed order into
// one write per gradient slot.
// Lists are walked back to front from T_final, recovering T_k = T_{k+1} /
// (1 - alpha_k), with the sum S the later entries contribute growing from
// zero. A segment of a split list but its last starts from the state the
// forward recorded at its end: T and S = G . (C_final - C_boundary).
// Bound by the vector ALU (about 55 instructions per used entry and wave, half
// of the launch) and by the waves' uneven shares of a round. With the records
// staged through LDS and 16-entry batches (56 KB of LDS, three workgroups per
// CU instead of five) one 640x480 view of 157k intersections took 88 us, now
// 71; 774k intersections 359, now 315; a view through a volume 207, now 141;
// eight 320x240 views with 986k (lists up to 2460) 613, now 530. Five waves per
// SIMD spill 18 registers; four spill none: 71, 306, 157 and 529 us.
//
// The second moments are sums of terms up to 60 times their result for specks
// away from the tile's corner, in FP32: they carry rounding of 1e-5 of their
// gradient's norm, which any change of the last bits of T, of the segments or
// of the order of these sums redraws. Moments about the tile's centre halve
// it, and up to 16 segments of equal length take 286 us for the eight views, but
// both give other values than these.
template <int NF>
__global__ void __launch_bounds__(kTilePix) __attribute__((amdgpu_waves_per_eu(5))) k_blend_bwd(RenderConst rc, const ViewDev* __restrict__ views,
                                                        char* ctx, CtxLayout L, asgs_images dout) {
  constexpr int CS = 4 + NF;
  constexpr int GS = 6 + CS;
  constexpr int NW = kTilePix / 64;
  constexpr int CP = 64;          // row of 64 pixel coefficients (bf16), 8-pixel groups XOR-swizzled by row
  constexpr int C1 = CS - 4;      // the second column block holds the last four channels and the moments
  // The first n_views kSplitPerView (kSegMax - 1) workgroups take the
  // segments but the last of the split lists, one split-record slot each
  // (and exit at once where there is none), the rest one blend position each
  // (longest lists first): the whole list, or its last segment.
  const uint32_t extra = (uint32_t)rc.n_views * kSplitPerView * (kSegMax - 1);
  const bool front = blockIdx.x < extra;
  uint4 bi;
  int nseg = 1, seg = 0;
  if (front) {
    bi = ctx_ptr<const uint4>(ctx, L.sinfo)[blockIdx.x / (kSegMax - 1)];
    if (bi.x == ~0u) return;
    nseg = split_segments(bi.z - bi.y);
    seg = (int)(blockIdx.x % (kSegMax - 1));
    if (seg >= nseg - 1) return;
  } else {
    bi = ctx_ptr<const uint4>(ctx, L.binfo)[blockIdx.x - extra];
    if (ctx_ptr<const uint32_t>(ctx, L.bslot)[bi.x]) nseg = split_segments(bi.z - bi.y);
    seg = nseg - 1;
  }
  // this workgroup's segment: entries [elo, eend) of the list
  const int elo = seg * kSeg, eend = front ? elo + kSeg : (int)(bi.z - bi.y);
  const int tile = (int)bi.x;
  const int view = find_view(views, rc.n_views, tile);
  const ViewDev& V = views[view];
  const int lt = tile - V.tile_base;
  const int ty = lt / V.TX, tx = lt - ty * V.TX;
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int x0 = tx * kTile, y0 = ty * kTile;
  const int px = x0 + tile_lx(t);
  const int py = y0 + tile_ly(t);
  const bool inside = px < V.W && py < V.H;
  const float pxf = (float)px, pyf = (float)py;
  const uint2 rg = make_uint2(bi.y, bi.z);
  prioritise(blockIdx.x, rc.n_cu);
  const uint32_t* pairgid = ctx_ptr<const uint32_t>(ctx, L.pairgid) + rg.x;
  const uint32_t* pslot = ctx_ptr<const uint32_t>(ctx, L.pslot) + rg.x;
  const float* geom = ctx_ptr<const float>(ctx, L.geom);
  const float* chan = ctx_ptr<const float>(ctx, L.chan);
  const uint8_t* pmask = ctx_ptr<const uint8_t>(ctx, L.pmask) + rg.x;
  float* gslot = ctx_ptr<float>(ctx, L.gslot);

  constexpr int kRound = 32;         // list entries per round (one per lane of half a wave)
  constexpr int PS = (GS + 3) & ~3;  // row of a partial-sum entry and of a gradient slot (whole float4)
  // per wave: 16 rows (w of 8 batch positions, then their dL/dpower) of 64
  // pixels, as bf16 hi and lo (before the first batch the array holds each
  // wave's channel gradients for the exchange into the MFMA operand layout)
  __shared__ __attribute__((aligned(16))) uint16_t acf[NW][2][2 * kBwdBatch][CP];
  __shared__ __attribute__((aligned(16))) float part[NW][kRound][PS];  // per wave: rows of its used entries, in walking order
  static_assert(kRound % kBwdBatch == 0, "whole batches of rows");
  __shared__ uint32_t sused[NW];                                       // per wave: the round's entries with a row
  __shared__ uint32_t slast[NW];                                       // per wave: the last entry it uses

  const size_t HW = (size_t)V.W * V.H;
  const size_t pb = (size_t)V.pix_base;
  float Tf = 1.f;
  uint32_t last = 0;
  float G[CS];
#pragma unroll
  for (int c = 0; c < CS; ++c) G[c] = 0.f;
  float GT = 0.f;
  if (inside) {
    const size_t pix = (size_t)py * V.W + px;
    Tf = ctx_ptr<const float>(ctx, L.tfinal)[pb + pix];
    last = ctx_ptr<const uint32_t>(ctx, L.ncontrib)[pb + pix];
    for (int c = 0; c < 3; ++c) G[c] = dout.rgb[3 * pb + c * HW + pix];
    G[3] = dout.depth[pb + pix];
#pragma unroll
    for (int c = 0; c < NF; ++c) G[4 + c] = dout.feat[NF * pb + c * HW + pix];
    const float ga = dout.alpha ? dout.alpha[pb + pix] : 0.f;
    GT = rc.bg[0] * G[0] + rc.bg[1] * G[1] + rc.bg[2] * G[2] - ga;
  }
  // the last entry any pixel of this wave, and of the workgroup, uses: entries
  // behind it are not walked
  uint32_t wlast = last;
  for (int o = 32; o > 0; o >>= 1) wlast = max(wlast, (uint32_t)__shfl_xor((int)wlast, o));
  if (lane == 0) slast[wv] = wlast;
  __syncthreads();
  const int ehi = min(eend, max(elo, (int)max(max(slast[0], slast[1]), max(slast[2], slast[3]))));
  const int whi = min(ehi, __builtin_amdgcn_readfirstlane((int)wlast));
  // The Gaussian ids and quarter masks of the first two rounds are requested
  // now, later rounds' two rounds ahead.
  int rhi = ehi, rlo = max(ehi - kRound, elo);  // entries [rlo, rhi) of the round
  // the round's ids and masks, lane l entry l
  auto ids = [&](int lo, int hi, uint32_t& g, uint32_t& m) {
    g = m = 0u;
    if (lane < hi - lo) {
      g = pairgid[lo + lane];
      m = pmask[lo + lane];
    }
  };
  uint32_t gidv, maskv, gidn, maskn;
  ids(rlo, rhi, gidv, maskv);
  int nlo = max(rlo - kRound, elo);  // start of the next round
  ids(nlo, rlo, gidn, maskn);
  // B operands of the MFMAs (v_mfma_f32_16x16x32_bf16): K block kb covers
  // pixels 32 kb .. 32 kb + 31 of this wave; lane l supplies column l % 16 of
  // pixels 32 kb + 8 (l / 16) + i, i = 0..7, split into bf16 hi + lo. Block 0
  // (with features): channels 0-15. Block 1: columns 0-3 the hi and 4-7 the lo
  // parts of the last four channels, columns 8-13 the pixel-coordinate moments
  // (exact in bf16). The gradients reach that layout through the wave's rows of LDS, 16
  // channels of 64 pixels at a time, each row's 4-pixel groups XOR-swizzled by
  // the row so that the 16 rows of one read fall in different banks.
  static_assert(sizeof(acf) / NW == 16 * 64 * 4, "exchange rows");
  float* gx = reinterpret_cast<float*>(&acf[wv][0][0][0]);
  const int fcol = lane & 15;
  bf8v b0h[2], b0l[2], b1[2];
  auto wave_sync = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto put = [&](int row, float v) { gx[row * 64 + ((((lane >> 2) ^ row) << 2) | (lane & 3))] = v; };
  auto get = [&](int row, int kb, float (&v)[8]) {
    const int q4 = 8 * kb + 2 * (lane >> 4);  // first 4-pixel group of the lane's 8 pixels in the wave
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float4 a = *reinterpret_cast<const float4*>(&gx[row * 64 + (((q4 + h) ^ row) << 2)]);
      v[4 * h] = a.x;
      v[4 * h + 1] = a.y;
      v[4 * h + 2] = a.z;
      v[4 * h + 3] = a.w;
    }
  };
  auto pack = [&](const float (&v)[8], bf8v& h, bf8v& l) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      uint16_t hi, lo;
      bf_split(v[i], hi, lo);
      h[i] = __builtin_bit_cast(__bf16, hi);
      l[i] = __builtin_bit_cast(__bf16, lo);
    }
  };
  if (NF > 0) {
#pragma unroll
    for (int c = 0; c < 16; ++c) put(c, G[c % CS]);
    wave_sync();
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      float v[8];
      get(fcol, kb, v);
      pack(v, b0h[kb], b0l[kb]);
    }
    wave_sync();
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) put(c, G[C1 + c]);
  wave_sync();
  // this lane's moment lx^ex ly^ey: pixel i of the lane's 8 lies at lx = lx0 + i, ly = ly0 + 4 kb
  const int ex = fcol == 9 || fcol == 12 ? 1 : fcol == 11 ? 2 : 0, ey = fcol == 10 || fcol == 12 ? 1 : fcol == 13 ? 2 : 0;
  const float cx0 = ex == 0 ? 1.f : 0.f, cx1 = ex == 1 ? 1.f : 0.f, cx2 = ex == 2 ? 1.f : 0.f;
  const float lx0 = (float)(8 * (wv & 1)), ly0 = (float)(8 * (wv >> 1) + (lane >> 4));
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    float v[8];
    get(fcol & 3, kb, v);
    const float fy = ly0 + (float)(4 * kb);
    const float my = fcol < 8 || fcol > 13 ? 0.f : ey == 0 ? 1.f : ey == 1 ? fy : fy * fy;
    const bool lo = fcol >= 4;  // columns 4-7: v - hi(v)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float fx = lx0 + (float)i;
      const float m = fmaf(fmaf(cx2, fx, cx1), fx, cx0) * my;
      const float h = __uint_as_float((uint32_t)bf_rne(v[i]) << 16);
      const float c = lo ? v[i] - h : v[i];
      b1[kb][i] = (__bf16)(fcol < 8 ? c : m);
    }
  }
  wave_sync();

  // entries behind every pixel's last Gaussian get zero gradient
  for (int q = ehi + t; q < eend; q += kTilePix) {
    float4* dst = reinterpret_cast<float4*>(gslot + (size_t)pslot[q] * PS);
#pragma unroll
    for (int c = 0; c < PS / 4; ++c) dst[c] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float T = Tf;
  float sacc = 0.f;  // sum over later Gaussians of w_l (G . c_l)
  if (front && inside && whi == eend) {
    // the state at the segment's end, recorded by the forward of this quarter if
    // it went so far: T there, and the later entries' sum. Where its pixels
    // stopped in an earlier segment it wrote none, and no pixel uses a later entry
    constexpr int SA = split_first(CS), SF = split_final(CS);
    const float* sp = ctx_ptr<const float>(ctx, L.split) + (size_t)(blockIdx.x / (kSegMax - 1)) * split_floats(CS);
    const float* rb = sp + ((size_t)seg * kTilePix + t) * SA;
    const float* rf = sp + (size_t)(kSegMax - 1) * kTilePix * SA + (size_t)t * SF;
    T = rb[0];
#pragma unroll
    for (int c = 0; c < CS; ++c) sacc = fmaf(G[c], rf[c] - rb[1 + c], sacc);
  }
  const float amax = rc.alpha_max;
  uint16_t* const ah = &acf[wv][0][0][0];
  uint16_t* const al = &acf[wv][1][0][0];
  int nb = 0, nrow = 0;  // batched entries; rows of the round already in part
  // Contract the wave's nb batched entries over its 64 pixels on the matrix
  // cores and store their rows of partial sums.
  auto flush = [&]() {
    // the coefficients are read back by other lanes of this wave only
    wave_sync();
    f4v d0 = {0.f, 0.f, 0.f, 0.f}, d1 = d0;
    // A operands: row l % 16, pixels 32 kb + 8 (l / 16) .. + 7
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const int p0 = (32 * kb + 8 * (lane >> 4)) ^ ((fcol & 7) << 3);
      const bf8v xh = *reinterpret_cast<const bf8v*>(&ah[fcol * CP + p0]);
      const bf8v xl = *reinterpret_cast<const bf8v*>(&al[fcol * CP + p0]);
      if (NF > 0) {
        d0 = mfma_bf(xh, b0h[kb], d0);
        d0 = mfma_bf(xh, b0l[kb], d0);
        d0 = mfma_bf(xl, b0h[kb], d0);
      }
      // columns 0-3: the low parts, from four lanes up; the others zero
      bf8v b1l;
      {
        typedef int i4v __attribute__((ext_vector_type(4)));
        const i4v src = __builtin_bit_cast(i4v, b1[kb]);
        i4v v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_update_dpp(0, src[i], 0x104, 0xF, 0x1, true);
        b1l = __builtin_bit_cast(bf8v, v);
      }
      d1 = mfma_bf(xh, b1[kb], d1);
      d1 = mfma_bf(xh, b1l, d1);
      d1 = mfma_bf(xl, b1[kb], d1);
    }
    // lane l holds column l % 16 of rows 4 (l / 16) + r: channels from the
    // rows of w (lanes 0-31), moments from the rows of dL/dpower
    const bool up = lane >= 32;
    const int col = up ? fcol - 8 : 6 + C1 + fcol;
    const bool keep = up ? (fcol >= 8 && fcol < 14) : fcol < 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // rows past a last batch of fewer than 8 entries belong to no entry and are not read
      float* row = part[wv][nrow + 4 * ((lane >> 4) & 1) + r];
      if (NF > 0 && !up) row[6 + fcol] = d0[r];
      if (keep) row[col] = d1[r];
    }
    nrow += kBwdBatch;
    nb = 0;
    wave_sync();  // the next batch overwrites the coefficients
  };
  // One entry: alpha and the channel dot product, the transmittance before
  // it, and its coefficients into the batch; entries no pixel of the wave
  // uses take no row.
  uint32_t used = 0u;
  auto entry = [&](const SRec<CS>& rec, int j) {
    float dx, dy;
    const float power = eval_power(rec.g[0], rec.g[1], rec.g[2], rec.g[3], rec.g[4], pxf, pyf, dx, dy);
    // same alpha threshold as the forward
    const bool use = (uint32_t)(rlo + j) < last && power <= 0.f && power >= rec.g[6];
    if (!any_lane(use)) return;
    used |= 1u << j;
    const float raw = rec.g[5] * __expf(power);
    const float alpha = fminf(amax, raw);
    const float ioma = __builtin_amdgcn_rcpf(1.f - alpha);
    float dot0 = 0.f, dot1 = 0.f;  // two independent chains
#pragma unroll
    for (int c = 0; c < CS; c += 2) {
      dot0 = fmaf(G[c], rec.ch(c), dot0);
      dot1 = fmaf(G[c + 1], rec.ch(c + 1), dot1);
    }
    const float dotg = dot0 + dot1;
    float wgt = 0.f, dpow = 0.f;
    const float Tk = T * ioma;
    const float w_ = alpha * Tk;
    const float dalpha = Tk * dotg - (sacc + GT * Tf) * ioma;
    if (use) {
      T = Tk;
      wgt = w_;
      sacc = fmaf(w_, dotg, sacc);
      dpow = raw < amax ? dalpha * alpha : 0.f;
    }
    const int sp = nb * CP + (lane ^ (nb << 3));  // swizzled position of this pixel in row nb
    uint16_t wh, wl, ph, pl;
    bf_split(wgt, wh, wl);
    bf_split(dpow, ph, pl);
    ah[sp] = wh;
    al[sp] = wl;
    ah[sp + kBwdBatch * CP] = ph;
    al[sp + kBwdBatch * CP] = pl;
    if (++nb == kBwdBatch) flush();
  };
  // the wave's entries of a round (those that can reach a pixel of its quarter)
  auto round_bits = [&]() -> uint32_t {
    return (uint32_t)__ballot(((maskv >> wv) & 1u) && rlo + lane < whi);
  };
  auto load = [&](SRec<CS>& r, int j) { r.load(geom, chan, (uint32_t)__builtin_amdgcn_readlane((int)gidv, j)); };
  auto top = [&](uint32_t b, int other) { return b ? 31 - __builtin_clz(b) : other; };
  while (rhi > rlo) {
    const int cnt = rhi - rlo;
    // the slot this thread's part of the round's sums goes to, and the entries
    // of the round after the next
    constexpr int F4 = PS / 4;
    const int re = t / F4, rf = t - re * F4;
    uint32_t rslot = 0u, gid2, mask2;
    if (re < cnt) rslot = pslot[rlo + re];
    const int lo2 = max(nlo - kRound, elo);
    ids(lo2, nlo, gid2, mask2);
    // the next round's records are touched now (a lane per entry, each wave
    // one of a record's cache lines), so that the scalar loads find them in
    // the L2
    float touch = 0.f;
    if (wv < (NF > 0 ? 3 : 2) && lane < rlo - nlo)
      touch = wv == 0 ? geom[(size_t)gidn * kGeomStride] : chan[(size_t)gidn * CS + (wv == 1 ? 0 : CS - 1)];
    used = 0u;
    nrow = 0;
    // each record is requested one entry ahead
    if (uint32_t bits = round_bits()) {
      SRec<CS> ra, rb;
      int j = top(bits, 0);
      load(ra, j);
      for (;;) {
        bits &= ~(1u << j);
        const int j2 = top(bits, j);
        load(rb, j2);
        entry(ra, j);
        if (!bits) break;
        bits &= ~(1u << j2);
        j = top(bits, j2);
        load(ra, j);
        entry(rb, j2);
        if (!bits) break;
      }
    }
    if (used) {
      // the conic, position and opacity parts of the wave's rows in closed form
      // from their moments (linear in them, so the four waves' rows still add
      // up), a row per lane; the records of its entries are requested before
      // the last batch is contracted
      const bool own = lane < kRound && ((used >> (lane & (kRound - 1))) & 1u);
      if (nb) flush();
      if (own) {
        const float4* gp = reinterpret_cast<const float4*>(geom + (size_t)gidv * kGeomStride);
        const float4 g0 = gp[0], g1 = gp[1];
        float* row = part[wv][__builtin_popcount((used >> lane) >> 1)];
        const float4 a = *reinterpret_cast<const float4*>(row);
        const float2 b = *reinterpret_cast<const float2*>(row + 4);
        const float M[6] = {a.x, a.y, a.z, a.w, b.x, b.y};
        const float uu = g0.x - (float)x0, vv = g0.y - (float)y0;  // tile-local centre
        const float Sdx = fmaf(uu, M[0], -M[1]);
        const float Sdy = fmaf(vv, M[0], -M[2]);
        const float Sxx = fmaf(uu * uu, M[0], -(2.f * uu * M[1])) + M[3];
        const float Sxy = fmaf(-vv, M[1], fmaf(uu * vv, M[0], -(uu * M[2]))) + M[4];
        const float Syy = fmaf(vv * vv, M[0], -(2.f * vv * M[2])) + M[5];
        *reinterpret_cast<float4*>(row) =
            make_float4(-fmaf(g0.w, Sdy, g0.z * Sdx), -fmaf(g0.w, Sdx, g1.x * Sdy), -0.5f * Sxx, -Sxy);
        *reinterpret_cast<float2*>(row + 4) = make_float2(-0.5f * Syy, M[0] / g1.y);
      }
    }
    if (lane == 0) sused[wv] = used;
    asm volatile("" ::"v"(touch));  // the touching load is kept, and waited for here
    __syncthreads();
    // the four waves' rows -> one gradient slot per entry, a float4 per thread
    static_assert(kRound * F4 <= kTilePix, "one float4 of a round's sums per thread");
    if (re < cnt) {
      float4 v[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        // a wave's rows are in walking order: entries above re come first
        const uint32_t u = sused[w];
        const int k = __builtin_popcount((u >> re) >> 1);
        const float4 a = reinterpret_cast<const float4*>(part[w][k])[rf];
        const bool has = (u >> re) & 1u;
        v[w] = make_float4(has ? a.x : 0.f, has ? a.y : 0.f, has ? a.z : 0.f, has ? a.w : 0.f);
      }
      reinterpret_cast<float4*>(gslot + (size_t)rslot * PS)[rf] =
          make_float4((v[0].x + v[1].x) + (v[2].x + v[3].x), (v[0].y + v[1].y) + (v[2].y + v[3].y),
                      (v[0].z + v[1].z) + (v[2].z + v[3].z), (v[0].w + v[1].w) + (v[2].w + v[3].w));
    }
    __syncthreads();
    rhi = rlo;
    rlo = nlo;
    gidv = gidn;
    maskv = maskn;
    nlo = lo2;
    gidn = gid2;
    maskn = mask2;
  }
}

}  // namespace

void launch_blend_forward(const RenderConst& rc, const CtxLayout& L, char* ctx, const asgs_images& out,
                          const BlendL1* l1, hipStream_t s) {
  const ViewDev* views = reinterpret_cast<const ViewDev*>(ctx + L.views);
  const BlendL1 a = l1 ? *l1 : BlendL1{};
  const dim3 grid((unsigned)((rc.total_tiles + 7) / 8 * 32));
  const dim3 block(64 * kFwdWaves);
  if (rc.nf == 16) {
    if (l1) hipLaunchKernelGGL((k_blend_fwd<16, true>), grid, block, 0, s, rc, views, ctx, L, out, a);
    else hipLaunchKernelGGL((k_blend_fwd<16, false>), grid, block, 0, s, rc, views, ctx, L, out, a);
  } else {
    if (l1) hipLaunchKernelGGL((k_blend_fwd<0, true>), grid, block, 0, s, rc, views, ctx, L, out, a);
    else hipLaunchKernelGGL((k_blend_fwd<0, false>), grid, block, 0, s, rc, views, ctx, L, out, a);
  }
}

void launch_l1_tile_loss(const RenderConst& rc, const CtxLayout& L, char* ctx, float* loss, hipStream_t s) {
  const ViewDev* views = reinterpret_cast<const ViewDev*>(ctx + L.views);
  hipLaunchKernelGGL(k_l1_tile_loss, dim3(rc.n_views), dim3(256), 0, s, views,
                     reinterpret_cast<const float*>(ctx + L.lpart), loss);
}

void launch_blend_backward(const RenderConst& rc, const CtxLayout& L, char* ctx, const asgs_images& dout,
                           hipStream_t s) {
  const ViewDev* views = reinterpret_cast<const ViewDev*>(ctx + L.views);
  if (rc.nf == 16)
    hipLaunchKernelGGL(k_blend_bwd<16>, dim3(rc.total_tiles + rc.n_views * kSplitPerView * (kSegMax - 1)),
                       dim3(kTilePix), 0, s, rc,
                       views, ctx, L,
                       dout);
  else
    hipLaunchKernelGGL(k_blend_bwd<0>, dim3(rc.total_tiles + rc.n_views * kSplitPerView * (kSegMax - 1)),
                       dim3(kTilePix), 0, s, rc,
                       views, ctx, L,
                       dout);
}

}  // namespace asgs
