// Launch of the products of a layer and of the head.  Every epilogue (and kernel family) is compiled in
// source files of its own.
#ifndef SV_PRODUCTS_H
#define SV_PRODUCTS_H

#include "sv_gemm_mid.h"
#include "sv_gemm_skinny.h"
#include "sv_gemm_thin.h"

namespace sv {

// (the numbers that sv_product_plan reports)
enum ProductKernel { PRODUCT_SKINNY = 0, PRODUCT_MID = 1, PRODUCT_THIN = 2 };
// How one product [M, K] x [N, K]^T is split over the chip.
struct ProductPlan {
  ProductKernel kernel;
  int rb, nt;                // row blocks (PRODUCT_THIN: half of one) and tiles of the kernel instance
  int lgS, gpx, m_tiles;     // K slices, column groups per XCD, blocks of rows
  int wg_x;                  // workgroups per XCD
  int unit_stride;           // float4 of exchange scratch per workgroup
  int planes, n_planes;      // EPI_RESID: row-sum planes per column group, in all
};
ProductPlan plan_product(int M, int N, int K, int wf, int n_xcd);
ProductPlan plan_head(int M, int N, int K, int n_xcd);     // EPI_OUT on bf16 weights

// Where a product finds its scratch.
struct ProductScratch {
  f32x4_t* xch;
  unsigned* group_cnt;
  int* status;
};

// epi: EPI_*; wf: weight format (0 bf16, 1 E4M3, 2 int4; EPI_OUT: 0 only)
void launch_product(const ProductPlan& p, int epi, int wf, int n_xcd, const uint4* Xs, const uint4* Wp, int N, int K,
                    const ProductScratch& s, const EpiArgs& e, hipStream_t st);

// one function per kernel family and epilogue, each in its own source file (skinny: rb = 0 is gemm_thin)
void launch_skinny_qkv(const SkinnyArgs& a, int rb, int nt, int wf, dim3 grid, hipStream_t st);
void launch_skinny_resid(const SkinnyArgs& a, int rb, int nt, int wf, dim3 grid, hipStream_t st);
void launch_skinny_swiglu(const SkinnyArgs& a, int rb, int nt, int wf, dim3 grid, hipStream_t st);
void launch_skinny_out(const SkinnyArgs& a, int rb, int nt, int wf, dim3 grid, hipStream_t st);
void launch_mid_qkv(const MidArgs& a, int rb, int nt, int wf, dim3 grid, hipStream_t st);
void launch_mid_resid(const MidArgs& a, int rb, int nt, int wf, dim3 grid, hipStream_t st);
void launch_mid_swiglu(const MidArgs& a, int rb, int nt, int wf, dim3 grid, hipStream_t st);
void launch_mid_out(const MidArgs& a, int rb, int nt, int wf, dim3 grid, hipStream_t st);

#define SV_INSTANTIATE_SKINNY(NAME, EPI, FORMATS)                                                              \
  template <int RB, int WF>                                                                                    \
  static void tiles(const SkinnyArgs& a, int nt, dim3 grid, hipStream_t st) {                                  \
    if (nt == 2) gemm_skinny<RB, 2, EPI, WF><<<grid, 256, 0, st>>>(a);                                         \
    else if (nt <= 4) gemm_skinny<RB, (RB > 2 ? 3 : 4), EPI, WF><<<grid, 256, 0, st>>>(a);                     \
    else if constexpr (RB <= 2) gemm_skinny<RB, 6, EPI, WF><<<grid, 256, 0, st>>>(a);                          \
  }                                                                                                            \
  template <int WF>                                                                                            \
  static void rows(const SkinnyArgs& a, int rb, int nt, dim3 grid, hipStream_t st) {                           \
    if (rb == 1) tiles<1, WF>(a, nt, grid, st);                                                                \
    else if (rb == 2) tiles<2, WF>(a, nt, grid, st);                                                           \
    else if (rb == 3) tiles<3, WF>(a, nt, grid, st);                                                           \
    else tiles<4, WF>(a, nt, grid, st);                                                                        \
  }                                                                                                            \
  template <int WF>                                                                                            \
  static void thin(const SkinnyArgs& a, int nt, dim3 grid, hipStream_t st) {                                   \
    if (nt == 2) gemm_thin<2, EPI, WF><<<grid, 256, 0, st>>>(a);                                               \
    else if (nt <= 4) gemm_thin<4, EPI, WF><<<grid, 256, 0, st>>>(a);                                          \
    else gemm_thin<6, EPI, WF><<<grid, 256, 0, st>>>(a);                                                       \
  }                                                                                                            \
  void NAME(const SkinnyArgs& a, int rb, int nt, int wf, dim3 grid, hipStream_t st) {                          \
    if (rb == 0) {                                                                                             \
      if (FORMATS > 2 && wf == 2) thin<(FORMATS > 2 ? 2 : 0)>(a, nt, grid, st);                                \
      else if (FORMATS > 1 && wf == 1) thin<(FORMATS > 1 ? 1 : 0)>(a, nt, grid, st);                           \
      else thin<0>(a, nt, grid, st);                                                                           \
    } else if (FORMATS > 2 && wf == 2) rows<(FORMATS > 2 ? 2 : 0)>(a, rb, nt, grid, st);                              \
    else if (FORMATS > 1 && wf == 1) rows<(FORMATS > 1 ? 1 : 0)>(a, rb, nt, grid, st);                         \
    else rows<0>(a, rb, nt, grid, st);                                                                         \
  }

#define SV_INSTANTIATE_MID(NAME, EPI, FORMATS)                                                                 \
  template <int RB, int WF>                                                                                    \
  static void tiles(const MidArgs& a, int nt, dim3 grid, hipStream_t st) {                                     \
    if (nt == 1) gemm_mid<RB, 1, EPI, WF><<<grid, 256, 0, st>>>(a);                                            \
    else if (nt == 2) gemm_mid<RB, 2, EPI, WF><<<grid, 256, 0, st>>>(a);                                       \
    else gemm_mid<RB, 3, EPI, WF><<<grid, 256, 0, st>>>(a);                                                    \
  }                                                                                                            \
  template <int WF>                                                                                            \
  static void rows(const MidArgs& a, int rb, int nt, dim3 grid, hipStream_t st) {                              \
    if (rb == 3) tiles<3, WF>(a, nt, grid, st);                                                                \
    else if (rb == 4) tiles<4, WF>(a, nt, grid, st);                                                           \
    else tiles<5, WF>(a, nt, grid, st);                                                                        \
  }                                                                                                            \
  void NAME(const MidArgs& a, int rb, int nt, int wf, dim3 grid, hipStream_t st) {                             \
    if (FORMATS > 2 && wf == 2) rows<(FORMATS > 2 ? 2 : 0)>(a, rb, nt, grid, st);                              \
    else if (FORMATS > 1 && wf == 1) rows<(FORMATS > 1 ? 1 : 0)>(a, rb, nt, grid, st);                         \
    else rows<0>(a, rb, nt, grid, st);                                                                         \
  }

}  // namespace sv
#endif
