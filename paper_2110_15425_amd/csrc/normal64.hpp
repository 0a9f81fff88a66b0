// normal64.hpp -- two standard normals in double from one Philox block.
//
// Box-Muller: rho = sqrt(-2 ln u_a), angle 2 pi u_b, with u = (m + 1) 2^-53 of
// a 53-bit word pair.  The arguments are known to be such multiples, so none
// of a general logarithm's or sine's special cases arise, and both functions
// come from a 128-entry table in LDS and a short polynomial:
//
//  * u_a = z 2^k with z in [0.6875, 1.375); entry i of z's 128 intervals holds
//    {-2 c 2^-53, T = 2 ln c} with c near 1 / z's interval centre, chosen so
//    that T, a multiple of 2^-43, is 2 ln c to 2^-61.  With q = 2 - 2 c z (one
//    fused multiply-add, |q| <= 2^-6),
//      -2 ln u_a = (T - 2 ln2 k) + q + q^2 Q(q),
//    the first term exact (2 ln2 is split into a multiple of 2^-43 and a rest).
//    c = 1 in the two intervals around z = 1, where the result is small, so
//    that it keeps its relative precision; their T is 10^-300, not 0, so that
//    u_a = 1 gives rho = 10^-150 instead of the square root of 0 by a
//    reciprocal.  The rounding of the last addition is carried as `err` into
//    the square root's residual.
//  * 2 pi u_b = 2 pi j / 128 + theta, |theta| <= 2 pi / 256: entry j holds
//    {cos, sin}(2 pi j / 128), theta's sine and cosine come from polynomials
//    (relative error below 2^-60), and the angle sum is folded into the
//    products with rho, so the table's value is never rounded again.
//
// Q and the two trigonometric polynomials are minimax fits (Remez) in 200-bit
// arithmetic.  v_rsq_f64 is good to 2^-24 (measured), hence one Newton step
// and one residual step.
//
// Bound by VALU issue.  Against the general log, sqrt and sincospi calls: 68
// instructions instead of 169; with them and the fused update a drift-diffusion
// sweep of 10^7 runs went from 4.45 to 2.23 ms, a 64 x 10^4 conflict sweep from
// 0.466 to 0.239 ms.  Mean error against an 80-bit evaluation 0.40 units in the
// last place (0.43 with the library calls).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include "internal.hpp"
#include "rng.hpp"

namespace cm {

struct alignas(16) NormPair {
  double a, b;
};
constexpr int kNormEntries = 128;
struct NormTab {
  NormPair log[kNormEntries];  // {-2 c 2^-53, 2 ln c}
  NormPair ang[kNormEntries];  // {cos, sin} of 2 pi j / 128
};
static_assert(sizeof(NormTab) == kNormTabBytes, "the launch plans count the table's LDS");

namespace {

constexpr NormTab kNormTabValues = {{
    {-0x1.734f0c53179d1p-52, 0x1.7cc7f7d86dc00p-1}, {-0x1.713786d9d7676p-52, 0x1.76feecb972800p-1},
    {-0x1.6f26016f33f4ap-52, 0x1.713e33a491000p-1}, {-0x1.6d1a6269104ffp-52, 0x1.6b85b4d2a6000p-1},
    {-0x1.6b1490ab38057p-52, 0x1.65d558d7b2000p-1}, {-0x1.691473a8921e1p-52, 0x1.602d08af17800p-1},
    {-0x1.6719f3600936bp-52, 0x1.5a8cadbbc8400p-1}, {-0x1.6524f853acb1bp-52, 0x1.54f431b7a7400p-1},
    {-0x1.63356b88a455bp-52, 0x1.4f637ebb93400p-1}, {-0x1.614b368415e7ep-52, 0x1.49da7f3ea3c00p-1},
    {-0x1.5f6643428fb71p-52, 0x1.44591e0530c00p-1}, {-0x1.5d867c3ddd9b0p-52, 0x1.3edf463955c00p-1},
    {-0x1.5babcc647e0fep-52, 0x1.396ce359b7400p-1}, {-0x1.59d61f124a64ap-52, 0x1.3401e12b15000p-1},
    {-0x1.580560159012bp-52, 0x1.2e9e2bce41000p-1}, {-0x1.56397ba7c99e8p-52, 0x1.2941afb194000p-1},
    {-0x1.54725e6cadffdp-52, 0x1.23ec5994cf000p-1}, {-0x1.52aff569888f2p-52, 0x1.1e9e16759c800p-1},
    {-0x1.50f22e10357ddp-52, 0x1.1956d3b6fec00p-1}, {-0x1.4f38f62dd7949p-52, 0x1.14167ef370000p-1},
    {-0x1.4d843bedc9991p-52, 0x1.0edd060b8d000p-1}, {-0x1.4bd3edd982744p-52, 0x1.09aa572ba5000p-1},
    {-0x1.4a27fad8505e5p-52, 0x1.047e60d0d1800p-1}, {-0x1.4880522014c62p-52, 0x1.feb2233ea2000p-2},
    {-0x1.46dce345914b9p-52, 0x1.f474b134c1800p-2}, {-0x1.453d9e2c82fcfp-52, 0x1.ea4449f093800p-2},
    {-0x1.43a2730acbbf0p-52, 0x1.e020cc6287000p-2}, {-0x1.420b5265e7f84p-52, 0x1.d60a17f912800p-2},
    {-0x1.40782d11b7fa3p-52, 0x1.cc000ca2ef800p-2}, {-0x1.3ee8f42985333p-52, 0x1.c2028aac23000p-2},
    {-0x1.3d5d991b87b61p-52, 0x1.b81173112a000p-2}, {-0x1.3bd60d9240cfbp-52, 0x1.ae2ca6f6cf000p-2},
    {-0x1.3a524387a4311p-52, 0x1.a454082e34800p-2}, {-0x1.38d22d357deabp-52, 0x1.9a8778d8ef000p-2},
    {-0x1.3755bd1bc13f0p-52, 0x1.90c6db9a5f000p-2}, {-0x1.35dce5f91ec65p-52, 0x1.8712136f96000p-2},
    {-0x1.34679acedce2fp-52, 0x1.7d6903d0a8800p-2}, {-0x1.32f5ced698b7fp-52, 0x1.73cb9074c0000p-2},
    {-0x1.3187758dc06a3p-52, 0x1.6a399da5eb000p-2}, {-0x1.301c82ab7efe5p-52, 0x1.60b31005f4800p-2},
    {-0x1.2eb4ea1fe0b1bp-52, 0x1.5737cc8fc5000p-2}, {-0x1.2d50a012dd303p-52, 0x1.4dc7b897f3800p-2},
    {-0x1.2bef98e5a97bfp-52, 0x1.4462b9dcc4800p-2}, {-0x1.2a91c92f3542bp-52, 0x1.3b08b67550800p-2},
    {-0x1.293725bb7543ep-52, 0x1.31b994d359000p-2}, {-0x1.27dfa38a0d422p-52, 0x1.28753bc0ae800p-2},
    {-0x1.268b37cd68142p-52, 0x1.1f3b925f5d800p-2}, {-0x1.2539d7e850aedp-52, 0x1.160c801f46000p-2},
    {-0x1.23eb7970b5497p-52, 0x1.0ce7ecd784000p-2}, {-0x1.22a01229f39e4p-52, 0x1.03cdc0a4bf800p-2},
    {-0x1.2157980556dc9p-52, 0x1.f57bc7e496000p-3}, {-0x1.2012011f40aa8p-52, 0x1.e3707ed764000p-3},
    {-0x1.1ecf43c7344aap-52, 0x1.d1797876fc000p-3}, {-0x1.1d8f5672dc0d5p-52, 0x1.bf96876981000p-3},
    {-0x1.1c522fc1caa4ep-52, 0x1.adc77ee57e000p-3}, {-0x1.1b17c67f2cf88p-52, 0x1.9c0c32d4e5000p-3},
    {-0x1.19e0119d35e68p-52, 0x1.8a64779d95000p-3}, {-0x1.18ab08383b541p-52, 0x1.78d022587a000p-3},
    {-0x1.1778a1926f719p-52, 0x1.674f089d97000p-3}, {-0x1.1648d50fd0f86p-52, 0x1.55e10051ac000p-3},
    {-0x1.151b9a3fd9fafp-52, 0x1.4485e03d8c000p-3}, {-0x1.13f0e8d27a7a9p-52, 0x1.333d7f75ce000p-3},
    {-0x1.12c8b89ed23a6p-52, 0x1.2207b5c6f3000p-3}, {-0x1.11a3019a7b5b3p-52, 0x1.10e45b3d15000p-3},
    {-0x1.107fbbe00bcd7p-52, 0x1.ffa6911a1c000p-4}, {-0x1.0f5edfabe6769p-52, 0x1.dda8addbbc000p-4},
    {-0x1.0e4065582964cp-52, 0x1.bbcebfc6f6000p-4}, {-0x1.0d2445641a8cap-52, 0x1.9a187b6e26000p-4},
    {-0x1.0c0a7868b1298p-52, 0x1.788595a2fe000p-4}, {-0x1.0af2f723a1cb6p-52, 0x1.5715c4d5b2000p-4},
    {-0x1.09ddba6aef490p-52, 0x1.35c8bfa900000p-4}, {-0x1.08cabb375d8dfp-52, 0x1.149e3e40e4000p-4},
    {-0x1.07b9f29b7ffc5p-52, 0x1.e72bf27dac000p-5}, {-0x1.06ab59c79a49dp-52, 0x1.a55f548e94000p-5},
    {-0x1.059eea0723a10p-52, 0x1.63d61785a8000p-5}, {-0x1.04949cc0c56cep-52, 0x1.228fb1d720000p-5},
    {-0x1.038c6b7782cdfp-52, 0x1.c31737fcb8000p-6}, {-0x1.02864fc6b6b26p-52, 0x1.41929f3978000p-6},
    {-0x1.018243645c238p-52, 0x1.8121208b20000p-7}, {-0x1.0000000000000p-52, 0x1.56e1fc2f8f359p-997},
    {-0x1.0000000000000p-52, 0x1.56e1fc2f8f359p-997}, {-0x1.fa11caa02a049p-53, -0x1.7dc475f570000p-6},
    {-0x1.f6310aca049bbp-53, -0x1.3cea443594000p-5}, {-0x1.f25f644399d40p-53, -0x1.b9fc024c98000p-5},
    {-0x1.ee9c7f845631cp-53, -0x1.1b0d98926a000p-4}, {-0x1.eae807acf877bp-53, -0x1.58a5bae61c000p-4},
    {-0x1.e741aa5ac5b98p-53, -0x1.95c830d672000p-4}, {-0x1.e3a9179dc86cfp-53, -0x1.d276b8ad3e000p-4},
    {-0x1.e01e01e020bc6p-53, -0x1.0759835977000p-3}, {-0x1.dca01dca0bc85p-53, -0x1.253f62f04c000p-3},
    {-0x1.d92f2231ed1abp-53, -0x1.42edcbea38000p-3}, {-0x1.d5cac807638fap-53, -0x1.60658a9309000p-3},
    {-0x1.d272ca3e75339p-53, -0x1.7da766e33c000p-3}, {-0x1.cf26e5c309694p-53, -0x1.9ab4246d28000p-3},
    {-0x1.cbe6d960233d5p-53, -0x1.b78c82bad5000p-3}, {-0x1.c8b265ae6c2d4p-53, -0x1.d4313d7271000p-3},
    {-0x1.c5894d10d1f4cp-53, -0x1.f0a30c012e000p-3}, {-0x1.c26b539430679p-53, -0x1.06715126d9800p-2},
    {-0x1.bf583ee86b492p-53, -0x1.1478584669000p-2}, {-0x1.bc4fd65886389p-53, -0x1.2266f1909b000p-2},
    {-0x1.b951e2b2d26c0p-53, -0x1.303d71886f800p-2}, {-0x1.b65e2e3ab27d9p-53, -0x1.3dfc2b1492800p-2},
    {-0x1.b37484ac4cf13p-53, -0x1.4ba36f3f4b800p-2}, {-0x1.b094b31ecb69bp-53, -0x1.59338d93b7000p-2},
    {-0x1.adbe87fa7c9b8p-53, -0x1.66acd42171000p-2}, {-0x1.aaf1d2f889606p-53, -0x1.740f8f53d0800p-2},
    {-0x1.a82e6511dcc9ep-53, -0x1.815c0a19f7800p-2}, {-0x1.a5741075672adp-53, -0x1.8e928dee05800p-2},
    {-0x1.a2c2a87c4887dp-53, -0x1.9bb362e80d000p-2}, {-0x1.a01a019ef1f83p-53, -0x1.a8becfce34000p-2},
    {-0x1.9d79f177de74cp-53, -0x1.b5b519e341800p-2}, {-0x1.9ae24ea678c97p-53, -0x1.c2968552ff800p-2},
    {-0x1.9852f0d8ec092p-53, -0x1.cf6354e09c800p-2}, {-0x1.95cbb0be3a1c8p-53, -0x1.dc1bca0ab1800p-2},
    {-0x1.934c67f9b3eb2p-53, -0x1.e8c0252aa0000p-2}, {-0x1.90d4f11f0552ep-53, -0x1.f550a56a38800p-2},
    {-0x1.8e6527af03e4bp-53, -0x1.00e6c45afd000p-1}, {-0x1.8bfce8051894dp-53, -0x1.071b85ffa8000p-1},
    {-0x1.899c0f60173d0p-53, -0x1.0d46b579af000p-1}, {-0x1.87427bcbfc321p-53, -0x1.136870295c800p-1},
    {-0x1.84f00c2896f74p-53, -0x1.1980d2da64c00p-1}, {-0x1.82a4a0192a5bdp-53, -0x1.1f8ff9e1e4000p-1},
    {-0x1.80601804f0918p-53, -0x1.25960110ce800p-1}, {-0x1.7e225516a83c9p-53, -0x1.2b9303a8d3000p-1},
    {-0x1.7beb3922d61c5p-53, -0x1.31871c955f000p-1}, {-0x1.79baa6bb690bbp-53, -0x1.3772662beec00p-1},
    {-0x1.7790811abd694p-53, -0x1.3d54fa5937000p-1}, {-0x1.756cac211dd05p-53, -0x1.432ef29d7ec00p-1},
  }, {
    {0x1.0000000000000p+0, 0.0}, {0x1.ff621e3796d7ep-1, 0x1.91f65f10dd814p-5},
    {0x1.fd88da3d12526p-1, 0x1.917a6bc29b42cp-4}, {0x1.fa7557f08a517p-1, 0x1.2c8106e8e613ap-3},
    {0x1.f6297cff75cb0p-1, 0x1.8f8b83c69a60bp-3}, {0x1.f0a7efb9230d7p-1, 0x1.f19f97b215f1bp-3},
    {0x1.e9f4156c62ddap-1, 0x1.294062ed59f06p-2}, {0x1.e212104f686e5p-1, 0x1.58f9a75ab1fddp-2},
    {0x1.d906bcf328d46p-1, 0x1.87de2a6aea963p-2}, {0x1.ced7af43cc773p-1, 0x1.b5d1009e15cc0p-2},
    {0x1.c38b2f180bdb1p-1, 0x1.e2b5d3806f63bp-2}, {0x1.b728345196e3ep-1, 0x1.073879922ffeep-1},
    {0x1.a9b66290ea1a3p-1, 0x1.1c73b39ae68c8p-1}, {0x1.9b3e047f38741p-1, 0x1.30ff7fce17035p-1},
    {0x1.8bc806b151741p-1, 0x1.44cf325091dd6p-1}, {0x1.7b5df226aafafp-1, 0x1.57d69348ceca0p-1},
    {0x1.6a09e667f3bcdp-1, 0x1.6a09e667f3bcdp-1}, {0x1.57d69348ceca0p-1, 0x1.7b5df226aafafp-1},
    {0x1.44cf325091dd6p-1, 0x1.8bc806b151741p-1}, {0x1.30ff7fce17035p-1, 0x1.9b3e047f38741p-1},
    {0x1.1c73b39ae68c8p-1, 0x1.a9b66290ea1a3p-1}, {0x1.073879922ffeep-1, 0x1.b728345196e3ep-1},
    {0x1.e2b5d3806f63bp-2, 0x1.c38b2f180bdb1p-1}, {0x1.b5d1009e15cc0p-2, 0x1.ced7af43cc773p-1},
    {0x1.87de2a6aea963p-2, 0x1.d906bcf328d46p-1}, {0x1.58f9a75ab1fddp-2, 0x1.e212104f686e5p-1},
    {0x1.294062ed59f06p-2, 0x1.e9f4156c62ddap-1}, {0x1.f19f97b215f1bp-3, 0x1.f0a7efb9230d7p-1},
    {0x1.8f8b83c69a60bp-3, 0x1.f6297cff75cb0p-1}, {0x1.2c8106e8e613ap-3, 0x1.fa7557f08a517p-1},
    {0x1.917a6bc29b42cp-4, 0x1.fd88da3d12526p-1}, {0x1.91f65f10dd814p-5, 0x1.ff621e3796d7ep-1},
    {0.0, 0x1.0000000000000p+0}, {-0x1.91f65f10dd814p-5, 0x1.ff621e3796d7ep-1},
    {-0x1.917a6bc29b42cp-4, 0x1.fd88da3d12526p-1}, {-0x1.2c8106e8e613ap-3, 0x1.fa7557f08a517p-1},
    {-0x1.8f8b83c69a60bp-3, 0x1.f6297cff75cb0p-1}, {-0x1.f19f97b215f1bp-3, 0x1.f0a7efb9230d7p-1},
    {-0x1.294062ed59f06p-2, 0x1.e9f4156c62ddap-1}, {-0x1.58f9a75ab1fddp-2, 0x1.e212104f686e5p-1},
    {-0x1.87de2a6aea963p-2, 0x1.d906bcf328d46p-1}, {-0x1.b5d1009e15cc0p-2, 0x1.ced7af43cc773p-1},
    {-0x1.e2b5d3806f63bp-2, 0x1.c38b2f180bdb1p-1}, {-0x1.073879922ffeep-1, 0x1.b728345196e3ep-1},
    {-0x1.1c73b39ae68c8p-1, 0x1.a9b66290ea1a3p-1}, {-0x1.30ff7fce17035p-1, 0x1.9b3e047f38741p-1},
    {-0x1.44cf325091dd6p-1, 0x1.8bc806b151741p-1}, {-0x1.57d69348ceca0p-1, 0x1.7b5df226aafafp-1},
    {-0x1.6a09e667f3bcdp-1, 0x1.6a09e667f3bcdp-1}, {-0x1.7b5df226aafafp-1, 0x1.57d69348ceca0p-1},
    {-0x1.8bc806b151741p-1, 0x1.44cf325091dd6p-1}, {-0x1.9b3e047f38741p-1, 0x1.30ff7fce17035p-1},
    {-0x1.a9b66290ea1a3p-1, 0x1.1c73b39ae68c8p-1}, {-0x1.b728345196e3ep-1, 0x1.073879922ffeep-1},
    {-0x1.c38b2f180bdb1p-1, 0x1.e2b5d3806f63bp-2}, {-0x1.ced7af43cc773p-1, 0x1.b5d1009e15cc0p-2},
    {-0x1.d906bcf328d46p-1, 0x1.87de2a6aea963p-2}, {-0x1.e212104f686e5p-1, 0x1.58f9a75ab1fddp-2},
    {-0x1.e9f4156c62ddap-1, 0x1.294062ed59f06p-2}, {-0x1.f0a7efb9230d7p-1, 0x1.f19f97b215f1bp-3},
    {-0x1.f6297cff75cb0p-1, 0x1.8f8b83c69a60bp-3}, {-0x1.fa7557f08a517p-1, 0x1.2c8106e8e613ap-3},
    {-0x1.fd88da3d12526p-1, 0x1.917a6bc29b42cp-4}, {-0x1.ff621e3796d7ep-1, 0x1.91f65f10dd814p-5},
    {-0x1.0000000000000p+0, 0.0}, {-0x1.ff621e3796d7ep-1, -0x1.91f65f10dd814p-5},
    {-0x1.fd88da3d12526p-1, -0x1.917a6bc29b42cp-4}, {-0x1.fa7557f08a517p-1, -0x1.2c8106e8e613ap-3},
    {-0x1.f6297cff75cb0p-1, -0x1.8f8b83c69a60bp-3}, {-0x1.f0a7efb9230d7p-1, -0x1.f19f97b215f1bp-3},
    {-0x1.e9f4156c62ddap-1, -0x1.294062ed59f06p-2}, {-0x1.e212104f686e5p-1, -0x1.58f9a75ab1fddp-2},
    {-0x1.d906bcf328d46p-1, -0x1.87de2a6aea963p-2}, {-0x1.ced7af43cc773p-1, -0x1.b5d1009e15cc0p-2},
    {-0x1.c38b2f180bdb1p-1, -0x1.e2b5d3806f63bp-2}, {-0x1.b728345196e3ep-1, -0x1.073879922ffeep-1},
    {-0x1.a9b66290ea1a3p-1, -0x1.1c73b39ae68c8p-1}, {-0x1.9b3e047f38741p-1, -0x1.30ff7fce17035p-1},
    {-0x1.8bc806b151741p-1, -0x1.44cf325091dd6p-1}, {-0x1.7b5df226aafafp-1, -0x1.57d69348ceca0p-1},
    {-0x1.6a09e667f3bcdp-1, -0x1.6a09e667f3bcdp-1}, {-0x1.57d69348ceca0p-1, -0x1.7b5df226aafafp-1},
    {-0x1.44cf325091dd6p-1, -0x1.8bc806b151741p-1}, {-0x1.30ff7fce17035p-1, -0x1.9b3e047f38741p-1},
    {-0x1.1c73b39ae68c8p-1, -0x1.a9b66290ea1a3p-1}, {-0x1.073879922ffeep-1, -0x1.b728345196e3ep-1},
    {-0x1.e2b5d3806f63bp-2, -0x1.c38b2f180bdb1p-1}, {-0x1.b5d1009e15cc0p-2, -0x1.ced7af43cc773p-1},
    {-0x1.87de2a6aea963p-2, -0x1.d906bcf328d46p-1}, {-0x1.58f9a75ab1fddp-2, -0x1.e212104f686e5p-1},
    {-0x1.294062ed59f06p-2, -0x1.e9f4156c62ddap-1}, {-0x1.f19f97b215f1bp-3, -0x1.f0a7efb9230d7p-1},
    {-0x1.8f8b83c69a60bp-3, -0x1.f6297cff75cb0p-1}, {-0x1.2c8106e8e613ap-3, -0x1.fa7557f08a517p-1},
    {-0x1.917a6bc29b42cp-4, -0x1.fd88da3d12526p-1}, {-0x1.91f65f10dd814p-5, -0x1.ff621e3796d7ep-1},
    {0.0, -0x1.0000000000000p+0}, {0x1.91f65f10dd814p-5, -0x1.ff621e3796d7ep-1},
    {0x1.917a6bc29b42cp-4, -0x1.fd88da3d12526p-1}, {0x1.2c8106e8e613ap-3, -0x1.fa7557f08a517p-1},
    {0x1.8f8b83c69a60bp-3, -0x1.f6297cff75cb0p-1}, {0x1.f19f97b215f1bp-3, -0x1.f0a7efb9230d7p-1},
    {0x1.294062ed59f06p-2, -0x1.e9f4156c62ddap-1}, {0x1.58f9a75ab1fddp-2, -0x1.e212104f686e5p-1},
    {0x1.87de2a6aea963p-2, -0x1.d906bcf328d46p-1}, {0x1.b5d1009e15cc0p-2, -0x1.ced7af43cc773p-1},
    {0x1.e2b5d3806f63bp-2, -0x1.c38b2f180bdb1p-1}, {0x1.073879922ffeep-1, -0x1.b728345196e3ep-1},
    {0x1.1c73b39ae68c8p-1, -0x1.a9b66290ea1a3p-1}, {0x1.30ff7fce17035p-1, -0x1.9b3e047f38741p-1},
    {0x1.44cf325091dd6p-1, -0x1.8bc806b151741p-1}, {0x1.57d69348ceca0p-1, -0x1.7b5df226aafafp-1},
    {0x1.6a09e667f3bcdp-1, -0x1.6a09e667f3bcdp-1}, {0x1.7b5df226aafafp-1, -0x1.57d69348ceca0p-1},
    {0x1.8bc806b151741p-1, -0x1.44cf325091dd6p-1}, {0x1.9b3e047f38741p-1, -0x1.30ff7fce17035p-1},
    {0x1.a9b66290ea1a3p-1, -0x1.1c73b39ae68c8p-1}, {0x1.b728345196e3ep-1, -0x1.073879922ffeep-1},
    {0x1.c38b2f180bdb1p-1, -0x1.e2b5d3806f63bp-2}, {0x1.ced7af43cc773p-1, -0x1.b5d1009e15cc0p-2},
    {0x1.d906bcf328d46p-1, -0x1.87de2a6aea963p-2}, {0x1.e212104f686e5p-1, -0x1.58f9a75ab1fddp-2},
    {0x1.e9f4156c62ddap-1, -0x1.294062ed59f06p-2}, {0x1.f0a7efb9230d7p-1, -0x1.f19f97b215f1bp-3},
    {0x1.f6297cff75cb0p-1, -0x1.8f8b83c69a60bp-3}, {0x1.fa7557f08a517p-1, -0x1.2c8106e8e613ap-3},
    {0x1.fd88da3d12526p-1, -0x1.917a6bc29b42cp-4}, {0x1.ff621e3796d7ep-1, -0x1.91f65f10dd814p-5},
  }};

// One copy per translation unit and device, read by the workgroups that stage
// it in LDS (and directly where a thread draws only once).
__device__ const NormTab kNormTab = kNormTabValues;

// Copies the table into LDS; the caller's next barrier makes it visible.
__device__ __forceinline__ void load_norm_tab(NormTab& t) {
  const NormPair* src = (const NormPair*)&kNormTab;
  NormPair* dst = (NormPair*)&t;
  for (uint32_t i = threadIdx.x; i < 2u * kNormEntries; i += blockDim.x) dst[i] = src[i];
}

// A kernel's table in LDS: nothing where the precision draws float normals.
template <int PREC>
struct NormLds {
  NormTab t;
  __device__ __forceinline__ void load() { load_norm_tab(t); }
  __device__ __forceinline__ const NormTab* get() const { return &t; }
};
struct NormNone {
  __device__ __forceinline__ void load() {}
  __device__ __forceinline__ const NormTab* get() const { return nullptr; }
};
template <>
struct NormLds<CM_FP32_STEP> : NormNone {};
template <>
struct NormLds<CM_BF16_PROJ> : NormNone {};

__host__ __device__ __forceinline__ uint64_t double_bits(double v) {
  uint64_t u;
  memcpy(&u, &v, 8);
  return u;
}
__host__ __device__ __forceinline__ double bits_double(uint64_t u) {
  double v;
  memcpy(&v, &u, 8);
  return v;
}

// a b + c with the polynomial coefficient c kept in registers of its own: left
// to itself the compiler copies every coefficient into the accumulator of a
// two-operand multiply-add, one more instruction for each.
__host__ __device__ __forceinline__ double fma_coef(double a, double b, double c) {
#ifdef __HIP_DEVICE_COMPILE__
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
#else
  return __builtin_fma(a, b, c);
#endif
}

// rsq(x): an approximation of 1 / sqrt(x) to about 2^-24.
template <class Rsq>
__host__ __device__ __forceinline__ void normals64_with(const Words& w, const NormTab& tab, Rsq rsq,
                                                        double& z0, double& z1) {
  // v = m + 1 in [1, 2^53], exactly; k and z from its bits
  const uint32_t top = w.w1 >> 11, bot = (w.w1 << 21) | (w.w0 >> 11);
  const double v = __builtin_fma((double)top, 4294967296.0, (double)bot) + 1.0;
  const uint64_t vb = double_bits(v);
  const uint32_t hi = (uint32_t)(vb >> 32), off = hi - 0x43360000u;  // 0.6875 2^53's high word
  const NormPair lt = tab.log[(off >> 13) & (kNormEntries - 1u)];
  const double kd = (double)((int32_t)off >> 20);
  const double z = bits_double(((uint64_t)(hi - (off & 0xFFF00000u)) << 32) | (uint32_t)vb);  // z 2^53
  const double q = __builtin_fma(z, lt.a, 2.0);
  const double s = __builtin_fma(kd, -0x1.62e42fefa3a00p+0, lt.b);  // exact
  double p = fma_coef(q, 0x1.249965b7141b8p-9, 0x1.555b556c88df3p-8);
  p = fma_coef(q, p, 0x1.99999988b5a59p-7);
  p = fma_coef(q, p, 0x1.fffffff6ffd00p-6);
  p = fma_coef(q, p, 0x1.55555555555abp-4);
  p = fma_coef(q, p, 0x1.0000000000008p-2);
  const double r = __builtin_fma(q * q, p, __builtin_fma(kd, 0x1.0ca86c3898d00p-48, q));
  const double x = s + r, err = (s - x) + r;  // |s| >= |r| or s = 10^-300
  const double y = rsq(x);
  const double h = 0.5 * y;
  double g = x * y;
  g = __builtin_fma(g, __builtin_fma(-g, h, 0.5), g);
  const double rho = __builtin_fma(__builtin_fma(-g, g, x) + err, h, g);
  // u_b: j the nearest of 128 parts of the circle, d the rest in 2^-53 revolutions
  const NormPair cs = tab.ang[(w.w3 + 0x01000000u) >> 25];
  const double d =
      __builtin_fma((double)((int32_t)(w.w3 << 7) >> 18), 4294967296.0, (double)((w.w3 << 21) | (w.w2 >> 11))) + 1.0;
  const double t = d * d;
  double sn = fma_coef(t, -0x1.32d17c6ea4e6dp-365, 0x1.466bc67688639p-259);
  sn = fma_coef(t, sn, -0x1.4abbce625be4dp-154);
  sn = d * fma_coef(t, sn, 0x1.921fb54442d18p-51);
  double cn = fma_coef(t, -0x1.55d25e6cc6afbp-312, 0x1.03c1f0812e1fbp-206);
  cn = t * fma_coef(t, cn, -0x1.3bd3cc9be45dcp-102);  // cos - 1
  z0 = __builtin_fma(rho, cs.a, rho * __builtin_fma(cs.a, cn, -(cs.b * sn)));
  z1 = __builtin_fma(rho, cs.b, rho * __builtin_fma(cs.a, sn, cs.b * cn));
}

__device__ __forceinline__ void normals64(const Words& w, const NormTab& tab, double& z0, double& z1) {
  normals64_with(w, tab, [](double x) { return __builtin_amdgcn_rsq(x); }, z0, z1);
}

}  // namespace
// 53-bit uniform in (0, 1] from a word pair: ((hi:lo) >> 11) + 1, times 2^-53.
// Built from two exact int->double conversions (the value fits in 53 bits).
__device__ __forceinline__ double uniform53(uint32_t lo, uint32_t hi) {
  const uint32_t top = hi >> 11;                 // bits 52..32 of the 53-bit value
  const uint32_t bot = (hi << 21) | (lo >> 11);  // bits 31..0
  const double v = __dadd_rn(__dmul_rn((double)top, 4294967296.0), (double)bot);
  return __dmul_rn(__dadd_rn(v, 1.0), 0x1p-53);
}

// The same normals by the library's functions, for results that hold the states'
// last bits: rho = sqrt(-2 ln u_a), the angle as sincospi(2 u_b), whose argument
// reduction is exact.
__device__ __forceinline__ void normals64_lib(const Words& w, double& z0, double& z1) {
  const double ua = uniform53(w.w0, w.w1);
  const double ub = uniform53(w.w2, w.w3);
  const double rho = sqrt(__dmul_rn(-2.0, log(ua)));
  double s, c;
  sincospi(__dmul_rn(2.0, ub), &s, &c);
  z0 = __dmul_rn(rho, c);
  z1 = __dmul_rn(rho, s);
}

}  // namespace cm
