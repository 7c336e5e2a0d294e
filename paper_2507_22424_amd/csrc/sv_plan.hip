// How the products are split over the chip, and their launches (host code only).
#include <cstring>

#include "sv_products.h"

namespace sv {

// Up to 128 rows, up to 16 with half of the rows left out.  As many K slices as leave a group at most skinny_max_tiles tiles while groups x slices
// make one round of the chip: fewer groups mean that fewer workgroups read the activations.  A wave gets
// at least 64 k-values (four waves per slice).
// 4-bit weights have gemm_thin only where a wave has two of its steps of 64 k-values and more: its ring asks for four
// steps whatever there is.  One row, us of a layer, gemm_skinny / gemm_thin: H = 512 36.0 / 37.1, H = 1024 38.1 / 39.9;
// 7B, two steps and more everywhere, 70.0 / 67.1.  (The other formats' steps are half as deep: faster throughout.)
static ProductPlan plan_skinny(int M, int N, int K, int wf, int n_xcd) {
  const int tiles = N / kFragRows, tiles_x = ceil_div(tiles, n_xcd);
  ProductPlan p;
  memset(&p, 0, sizeof(p));
  p.rb = ceil_div(M, kFragRows);
  const int most = skinny_max_tiles(p.rb);
  int nt = 0;
  for (p.lgS = 3; p.lgS >= 0; --p.lgS) {
    p.gpx = kCusPerXcd >> p.lgS;
    if (p.gpx > tiles_x) p.gpx = tiles_x;
    nt = ceil_div(tiles, n_xcd * p.gpx);
    if (nt <= most && K >= (256 << p.lgS)) break;
  }
  if (p.lgS < 0) {
    p.lgS = 0;
    p.gpx = ceil_div(tiles_x, most);
    nt = ceil_div(tiles, n_xcd * p.gpx);
  }
  p.kernel = M <= kThinRows && (wf != 2 || K >= (512 << p.lgS)) ? PRODUCT_THIN : PRODUCT_SKINNY;
  p.nt = nt <= 2 ? 2 : (p.rb > 2 ? 3 : (nt <= 4 ? 4 : 6));
  p.m_tiles = 1;
  p.wg_x = p.gpx << p.lgS;
  p.unit_stride = kSkinnyUnitStride;
  p.planes = 0;
  p.n_planes = tiles;
  return p;
}

// gemm_mid: every (row blocks, tiles, slices) it has is priced and the cheapest taken.  Fitted to sweeps of
// all of them on the 7B shapes at 70 - 960 rows, so that what is taken is on average within 0.5 % of the fastest: with
// every CU busy a k-step takes RB * (0.036 * NT + 0.036) us (the second term: what does not depend on the tiles, LDS
// reads of the activations among it), at least what HBM takes for the weights; a round of workgroups adds 11.4 us
// around its loop and 0.13 us per KiB of sums a workgroup hands to the others.
static ProductPlan plan_mid(int M, int N, int K, int wf, int n_xcd) {
  const int tiles = N / kFragRows, tiles_x = ceil_div(tiles, n_xcd), n_rb = ceil_div(M, 32), nks = K / kFragK;
  const double w_bytes = (double)N * K * 2 / (1 << wf);
  ProductPlan best;
  memset(&best, 0, sizeof(best));
  double best_us = 1e30;
  for (int rb = 3; rb <= kMidMaxRows; ++rb)
    for (int nt = 1; nt <= kMidMaxTiles; ++nt)
      for (int lgS = 0; lgS <= 3; ++lgS) {
        // at least 128 k-values a slice (4-bit weights 256); 256 for 8-bit weights too, whose chunk is 64, cost H = 512,
        // 400 rows, 5 % of a layer (63.3 / 66.6 us)
        if (lgS > 0 && K < ((wf == 2 ? 256 : 128) << lgS)) continue;
        ProductPlan p;
        memset(&p, 0, sizeof(p));
        p.kernel = PRODUCT_MID; p.rb = rb; p.nt = nt; p.lgS = lgS;
        p.m_tiles = ceil_div(n_rb, rb);
        p.gpx = ceil_div(tiles_x, 4 * nt);
        p.wg_x = (p.gpx * p.m_tiles) << lgS;
        if (lgS > 0 && p.gpx * p.m_tiles > kMaxGroups / n_xcd) continue;
        const int rounds = ceil_div(p.wg_x, kCusPerXcd);
        const double steps = (double)nks / (1 << lgS), kib = 16.0 * rb * nt * ((1 << lgS) - 1) / (1 << lgS);
        double loop = rounds * steps * rb * (0.036 * nt + 0.036);
        const double hbm = w_bytes / 6.4e6;
        if (loop < hbm) loop = hbm;
        const double us = loop + rounds * (11.4 + 0.13 * kib);
        if (us < best_us) {
          best_us = us;
          best = p;
        }
      }
  best.unit_stride = mid_unit_stride(best.rb, best.nt);
  best.planes = mid_planes(best.rb, best.nt, best.lgS);
  const int groups = n_xcd * best.gpx;
  best.n_planes = (tiles < groups ? tiles : groups) * best.planes;
  return best;
}

// Rows the kernels split at.  Up to 16 gemm_thin, up to 64 gemm_skinny.  Up to 128 gemm_skinny unless its groups of few
// tiles would make more than one round of the chip, or read too much of the activations: a group reads all rows of its
// K slice, so those that do not split K and those of two tiles or less, with 3 bytes of activations and more to a byte
// of weights, wait for them.  bf16 weights, us of gemm_skinny / gemm_mid (blocks of 12 tiles and more) at 80 and 112
// rows: one slice: gate+up of H = 3072 34 / 28, 39 / 33, of 7B 52 / 45, 60 / 54, q,k,v of H = 8192 99 / 78, 115 / 93; two
// tiles: down of 7B (271 and 361 MB read) 32.0 / 30.0, 36.5 / 33.6, output of H = 8192 45.4 / 41.1, 52.6 / 47.8, but
// output of 7B (101, 134 MB) 17.3 / 18.8, 19.2 / 20.6, down of H = 2048 (69, 92 MB) 14.7 / 17.4, 16.4 / 18.8; hence the
// 250 MB.  Slices and more tiles: q,k,v of 7B 33.4 / 33.5, 37.7 / 39.0, down of H = 5120 47.0 / 47.8, 53.0 / 54.6, output of
// H = 6144 28.2 / 29.6, 32.1 / 33.6.  Over H = 512 .. 8192 (32 products, 65 - 128 rows) what is taken is nowhere more than
// 1 % slower than gemm_skinny.  Coded weights: gemm_mid is slower or the same but where there is one slice (8 bits,
// q,k,v of H = 5120 40 / 36), which was not taken up.
ProductPlan plan_product(int M, int N, int K, int wf, int n_xcd) {
  if (M <= kSkinnyMaxRows) {
    const ProductPlan p = plan_skinny(M, N, K, wf, n_xcd);
    const int groups = n_xcd * p.gpx;
    const double mb = (double)groups * K * p.rb * kFragRows * 4 / 1e6;       // activations read
    const bool wide = wf == 0 && mb > 250 && (p.lgS == 0 || N / kFragRows <= 2 * groups);
    if (M <= 64 || (p.wg_x <= kCusPerXcd && !wide)) return p;
  }
  return plan_mid(M, N, K, wf, n_xcd);
}

// The head's product of more than 64 rows and at most two weight tiles per XCD (the 256 action rows): gemm_skinny
// on blocks of rows, as many K slices and as few rows per workgroup as one round of the chip takes.  Elsewhere
// plan_product: of gemm_mid's four waves, three would have no tile here.  us of the whole call, 256 columns of
// H = 4096, without / with this at 65, 150, 240, 480, 960 rows: 16.1 / 14.7, 22.4 / 17.8, 24.6 / 21.0, 30.5 / 26.9,
// 39.6 / 35.9; H = 1024: 13.8 / 12.8, 16.6 / 14.0, 17.2 / 13.8, 19.0 / 16.0, 23.3 / 21.7; 512 columns: the same or
// up to 20 % less; from 1024 columns on: 10 % less to 11 % more.
// Up to 16 rows gemm_thin only where a wave has the four steps of 32 k-values that its ring asks for.  us of the call, 8
// rows, gemm_skinny / gemm_thin: H = 1024 (two steps) 256 columns 10.2 / 10.6, 1024 columns 10.6 / 11.1; H = 4096 (four)
// 11.7 / 11.2, 12.1 / 11.2; 32000 columns of H = 1024 (eight) 23.5 / 22.2.  (The layers' short products gain by it all the same:
// they exchange their sums more often.  One row, H = 512, a layer 36.4 / 34.6.)
ProductPlan plan_head(int M, int N, int K, int n_xcd) {
  const int tiles = N / kFragRows, tiles_x = ceil_div(tiles, n_xcd), n_rb = ceil_div(M, kFragRows);
  for (int lgS = 3; M > 64 && tiles_x <= 2 && lgS >= 0; --lgS) {
    if (K < (256 << lgS)) continue;
    for (int rb = 1; rb <= 4; ++rb) {
      const int m_tiles = ceil_div(n_rb, rb), fit = (kCusPerXcd >> lgS) / m_tiles, gpx = fit < tiles_x ? fit : tiles_x;
      if (gpx < 1) continue;
      const int nt = ceil_div(tiles, n_xcd * gpx);
      if (nt > skinny_max_tiles(rb)) continue;
      ProductPlan p;
      memset(&p, 0, sizeof(p));
      p.kernel = PRODUCT_SKINNY; p.rb = rb; p.lgS = lgS; p.gpx = gpx; p.m_tiles = m_tiles;
      p.nt = nt <= 2 ? 2 : (rb > 2 ? 3 : (nt <= 4 ? 4 : 6));
      p.wg_x = (gpx * m_tiles) << lgS;
      p.unit_stride = kSkinnyUnitStride;
      p.n_planes = tiles;
      return p;
    }
  }
  ProductPlan p = plan_product(M, N, K, 0, n_xcd);
  if (p.kernel == PRODUCT_THIN && K < (512 << p.lgS)) p.kernel = PRODUCT_SKINNY;
  return p;
}

void launch_product(const ProductPlan& p, int epi, int wf, int n_xcd, const uint4* Xs, const uint4* Wp, int N, int K,
                    const ProductScratch& s, const EpiArgs& e, hipStream_t st) {
  const int tiles = N / kFragRows, groups = n_xcd * p.gpx;
  const bool mid = p.kernel == PRODUCT_MID;
  const dim3 grid(n_xcd, mid ? p.wg_x : p.gpx << p.lgS, mid ? 1 : p.m_tiles);
  if (mid) {
    MidArgs a;
    memset(&a, 0, sizeof(a));
    const int chunks = K / mid_chunk_k(p.rb, p.nt, wf);
    a.Xs = Xs; a.Wp = Wp; a.N = N; a.lgS = p.lgS; a.gpx = p.gpx; a.n_xcd = n_xcd; a.m_tiles = p.m_tiles;
    a.tq = tiles / groups; a.trem = tiles % groups;
    a.cq = chunks >> p.lgS; a.crem = chunks & ((1 << p.lgS) - 1);
    a.planes = p.planes;
    a.xch = s.xch; a.group_cnt = s.group_cnt; a.status = s.status; a.ucap = p.wg_x; a.unit_stride = p.unit_stride;
    a.gcap = kMaxGroups / n_xcd;
    a.e = e;
    auto* launch = epi == EPI_QKV ? launch_mid_qkv : (epi == EPI_RESID ? launch_mid_resid : (epi == EPI_SWIGLU ? launch_mid_swiglu : launch_mid_out));
    launch(a, p.rb, p.nt, wf, grid, st);
  } else {
    SkinnyArgs a;
    memset(&a, 0, sizeof(a));
    const bool thin = p.kernel == PRODUCT_THIN;
    const int units = K / (thin ? thin_step_k(wf) : kFragK << wf), waves = 4 << p.lgS;
    a.Xs = Xs; a.Wp = Wp; a.N = N; a.lgS = p.lgS; a.gpx = p.gpx; a.n_xcd = n_xcd;
    // Groups end at half tiles where that makes the largest group smaller, the weight bytes set the time (up to
    // 32 rows of bf16 weights) and nothing is written per tile (the residual's row sums are).  7B, gate/up, 5.375 tiles
    // a group: single row 3247 -> 3185 us per step, one layer of 26 nodes 104.3 -> 102.7; 60 rows 3851 -> 3864, and 3 %
    // slower with 8-bit and 4-bit weights: more groups then multiply (and convert) six tiles.
    const bool halves = p.rb == 1 && wf == 0 && epi != EPI_RESID && ceil_div(2 * tiles, groups) % 2;
    a.lgH = halves ? 0 : 1;
    const int pieces = halves ? 2 * tiles : tiles;
    a.tq = pieces / groups; a.trem = pieces % groups;
    a.uq = units / waves; a.urem = units % waves;
    a.xch = s.xch; a.group_cnt = s.group_cnt; a.status = s.status; a.ucap = p.wg_x; a.unit_stride = p.unit_stride;
    a.gcap = kMaxGroups / n_xcd;
    a.e = e;
    auto* launch = epi == EPI_QKV ? launch_skinny_qkv : (epi == EPI_RESID ? launch_skinny_resid : (epi == EPI_SWIGLU ? launch_skinny_swiglu : launch_skinny_out));
    launch(a, thin ? 0 : p.rb, p.nt, wf, grid, st);
  }
}

}  // namespace sv
