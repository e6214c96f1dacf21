// Which block-solve kernel serves a call.  Host code only.
#pragma once

namespace dd {

enum { P64 = 0, P32 = 1, P16 = 2, PB16 = 3 };   // FP64, FP32, FP16, BF16 storage

// How a block-solve workgroup forms the SU(3) products of its hops:
// PRODUCT_LANE, one right-hand side per workgroup and one site per thread
// (VALU); the TILE forms take a tile of right-hand sides of one lattice per
// workgroup (4^4 domains, FP16 or BF16 storage) with the product on the VALU
// (two right-hand sides), on FP32 MFMA, or on BF16-input MFMA with FP32
// accumulation (four).
// PRODUCT_LANE_SPLIT, two threads per site, and PRODUCT_LANE_HALVES, one thread per
// site with the sums in the order of PRODUCT_LANE_SPLIT, are not selected by the
// caller: the functions below name them for PRODUCT_LANE.
enum { PRODUCT_LANE = 0, PRODUCT_TILE_VALU = 1, PRODUCT_TILE_MFMA_F32 = 2, PRODUCT_TILE_MFMA_BF16 = 3, PRODUCT_LANE_SPLIT = 4,
       PRODUCT_LANE_HALVES = 5 };

// Two threads per site (the split form) or one, for domains of `sites` sites and
// a lattice of `workgroups` workgroups a colour.
//
// 288 sites (6x6x2x4): always two.  One thread per site needs 320-thread
// workgroups whose parities share a wave, and is slower at every size (in FP32
// its registers spill, too): three cycles on 24^3x32 with 12 right-hand sides
// took 16.8 ms in FP32 and 12.5 in FP16 against 10.3 and 9.7, on 12^3x24 with one
// 404 and 310 us against 233 and 227.  It is not built.
// FP64 on 16 sites: two (78.6 against 681 us a launch on 16^3x32); FP64 on others:
// one, it has no other kernel.
// 512 sites have two waves per SIMD with one thread per site.
// Others: two where one would leave the device idle, a colour of at most one
// workgroup per CU.  At 256 workgroups of 4^4 domains two threads per site take
// 33.7 us and one takes 40.5; beyond, a second round of workgroups begins, while
// with one thread per site two workgroups share a CU.  The form fixes the order of
// the sums, so it looks at the lattice, not at the launch: a system is solved with
// the same bits alone and in a batch.
constexpr int SPLIT_MAX = 256;
constexpr int sap_kernel_form(int sites, int prec, int product, long workgroups)
{
    if (product != PRODUCT_LANE) return product;
    if (sites == 288) return PRODUCT_LANE_SPLIT;
    if (prec == P64) return sites == 16 ? PRODUCT_LANE_SPLIT : PRODUCT_LANE;
    return sites < 512 && workgroups <= SPLIT_MAX ? PRODUCT_LANE_SPLIT : PRODUCT_LANE;
}

// The kernel that a launch of `workgroups` workgroups in all, over systems of one
// form, takes.  Several systems of small lattices can fill the device, and then
// two threads per site of 4^4 domains lose what they gained: three cycles for
// 12 right-hand sides on 16^3x32 (3072 workgroups a colour) take 2.60 ms in FP32
// and 2.39 in FP16, with one thread per site and the same bits 2.14 and 1.98; for
// three on 16^4 (384 workgroups) 413 and 391 us against 359 and 342, for two (256)
// 228 and 223 against 302 and 293.  (One thread per site in its own order of sums:
// 1.88 and 1.84 ms, 325 and 323 us.)  16 sites: two workgroups of two threads per
// site share a CU, and 12 right-hand sides on 12^3x24 (1944 workgroups) take 874 us
// against 783 with one thread in its own order: no kernel for that; 288: see above.
constexpr int sap_launch_form(int sites, int form, long workgroups)
{
    return form == PRODUCT_LANE_SPLIT && sites == 256 && workgroups > SPLIT_MAX ? PRODUCT_LANE_HALVES : form;
}

}  // namespace dd
