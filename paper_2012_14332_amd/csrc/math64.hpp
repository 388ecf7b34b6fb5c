// Float64 elementary functions of the float64 paths, for the arguments these
// paths have: logarithms of positive normal numbers, sine and cosine of one
// turn, M^n of a count M >= 1, square roots and quotients in the middle of the
// exponent range. What the general library functions spend on arguments that
// cannot occur here (huge angles, subnormals, negative bases) and on repeated
// reductions is left out: a model day in float64 takes about 430 vector
// instructions with these and about 1000 with the library's.
//
// The logarithm and the exponential are table-driven in the manner of P. T. P. Tang
// (ACM Trans. Math. Software 16, 1990, 378-400, and 15, 1989, 144-157), the
// logarithm's remainder by a reciprocal from the table (W. F. Wong and E. Goto, IEEE
// Trans. Computers 43, 1994, 278-294); the angle is reduced as by Cody and Waite
// (Software Manual for the Elementary Functions, 1980); quotient and square root are
// one iteration and a residual correction (P. Markstein, IBM J. Res. Dev. 34, 1990,
// 111-119). The tables are the functions' own values split in two parts, the
// coefficients interpolations at Chebyshev nodes (sine, cosine) and plain Taylor
// terms (logarithm, exponential).
//
// Largest errors against 64-bit significands, in units of the last place of the
// result: logarithm 0.51, power 0.55, sine and cosine 0.78; square root and quotients
// are correctly rounded (0.500) with seeds as far off as their instructions may be.
// The tables (3.5 KB) are staged in LDS: they sit in the walk's dependency chain,
// where an LDS read is the shortest.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace abc {

// -ln(c) = hi + lo for c close to the reciprocal of the interval's centre
// (12 significant bits, so that z c - 1 loses nothing that matters). Entry i
// belongs to significands in [1 + i / 128, 1 + (i + 1) / 128), halved from
// i = 64 on, so that z is in [3/4, 3/2). The intervals at z = 1 have c = 1, so
// logarithms near zero keep their relative precision. hi is a multiple of
// 2^-42: e ln2_hi + hi is exact for |e| < 2^10.
struct LogEntry {
    double c, hi, lo;
};
constexpr int LOG_N = 128;
__device__ const LogEntry LOG_TABLE[LOG_N] = {
    {0x1.0000000000000p+0, 0x0.0p+0, 0x0.0p+0},
    {0x1.fa00000000000p-1, 0x1.82448a3880000p-7, 0x1.4554412c584e0p-44},
    {0x1.f640000000000p-1, 0x1.3b024b78c0000p-6, 0x1.59a5e23a02f83p-44},
    {0x1.f240000000000p-1, 0x1.be0422fcd0000p-6, 0x1.a3d8850fe5939p-44},
    {0x1.ee80000000000p-1, 0x1.1ce5a62bc0000p-5, 0x1.a9cc78d8df999p-44},
    {0x1.eb00000000000p-1, 0x1.5715c4c040000p-5, -0x1.8888ddfc47628p-44},
    {0x1.e740000000000p-1, 0x1.95e430f8d0000p-5, -0x1.ba22cf76874ddp-45},
    {0x1.e3c0000000000p-1, 0x1.d0f2c1dda8000p-5, -0x1.8e40e3ef1e888p-45},
    {0x1.e000000000000p-1, 0x1.08598b59e4000p-4, -0x1.7e5dd7009902cp-46},
    {0x1.dcc0000000000p-1, 0x1.242d6c1a58000p-4, 0x1.4b838ac648481p-45},
    {0x1.d940000000000p-1, 0x1.425bce8474000p-4, 0x1.365ac5219daefp-45},
    {0x1.d5c0000000000p-1, 0x1.60c38ba798000p-4, 0x1.45cb10ebb04a5p-44},
    {0x1.d280000000000p-1, 0x1.7d33687c28000p-4, 0x1.3c88c3e706706p-44},
    {0x1.cf40000000000p-1, 0x1.99d62a65ec000p-4, -0x1.a45d04f9775edp-46},
    {0x1.cc00000000000p-1, 0x1.b6ac88dad4000p-4, 0x1.b1bdff50225c7p-44},
    {0x1.c8c0000000000p-1, 0x1.d3b73f37e0000p-4, 0x1.f9a8099ed2804p-44},
    {0x1.c580000000000p-1, 0x1.f0f70cdd98000p-4, 0x1.2e31f6c272c1ep-44},
    {0x1.c280000000000p-1, 0x1.06135354d4000p-3, 0x1.6304628340ee9p-44},
    {0x1.bf40000000000p-1, 0x1.14e75b48a0000p-3, -0x1.03dcc900f371fp-51},
    {0x1.bc40000000000p-1, 0x1.22aff2ddbe000p-3, -0x1.a3c2a6b069620p-45},
    {0x1.b940000000000p-1, 0x1.3090733ce4000p-3, -0x1.819b90764f584p-45},
    {0x1.b640000000000p-1, 0x1.3e892fe996000p-3, -0x1.24aa9375956dcp-44},
    {0x1.b380000000000p-1, 0x1.4b6d6fefe2000p-3, 0x1.522ecf56e7952p-46},
    {0x1.b080000000000p-1, 0x1.59958ff1d6000p-3, -0x1.a1d059769ca05p-44},
    {0x1.adc0000000000p-1, 0x1.66a5d42a3a000p-3, 0x1.a68933aa00298p-44},
    {0x1.ab00000000000p-1, 0x1.73cb9074fe000p-3, -0x1.d66a90d0005a6p-44},
    {0x1.a840000000000p-1, 0x1.81070bd7ba000p-3, -0x1.ff00bfaccbe8dp-44},
    {0x1.a580000000000p-1, 0x1.8e588ebac2000p-3, 0x1.b7d5cab2d1140p-44},
    {0x1.a2c0000000000p-1, 0x1.9bc062f270000p-3, -0x1.e2c9f9fd864adp-46},
    {0x1.a000000000000p-1, 0x1.a93ed3c8ae000p-3, -0x1.8724350562169p-45},
    {0x1.9d80000000000p-1, 0x1.b5971a213a000p-3, 0x1.9b50e83aa91dfp-44},
    {0x1.9b00000000000p-1, 0x1.c2028ab180000p-3, -0x1.92e0ee55c7ac6p-45},
    {0x1.9840000000000p-1, 0x1.cfc25714be000p-3, -0x1.810b32c7f1bbep-46},
    {0x1.95c0000000000p-1, 0x1.dc56cae452000p-3, 0x1.eb37aa24e1817p-44},
    {0x1.9340000000000p-1, 0x1.e8ff2622ba000p-3, 0x1.78e13d33981e5p-44},
    {0x1.90c0000000000p-1, 0x1.f5bba83060000p-3, 0x1.41b254a43da63p-44},
    {0x1.8e80000000000p-1, 0x1.00a1c6adda000p-2, 0x1.1cd8d688b9e18p-44},
    {0x1.8c00000000000p-1, 0x1.07138604d6000p-2, -0x1.e76324e912b17p-44},
    {0x1.8980000000000p-1, 0x1.0d8fb813eb000p-2, 0x1.ee8c88753fa35p-46},
    {0x1.8740000000000p-1, 0x1.136ef02e83000p-2, -0x1.bd05830e58250p-44},
    {0x1.8500000000000p-1, 0x1.1956d3b9bc000p-2, 0x1.7d2f73ad1aa14p-45},
    {0x1.82c0000000000p-1, 0x1.1f477c7573000p-2, 0x1.6d6d4010d751ap-45},
    {0x1.8080000000000p-1, 0x1.25410494e5000p-2, 0x1.b1d7ac0ef77f2p-44},
    {0x1.7e40000000000p-1, 0x1.2b4386c169000p-2, -0x1.e7d8c5cbc9cf9p-47},
    {0x1.7c00000000000p-1, 0x1.314f1e1d36000p-2, -0x1.8e27ad3213cb8p-45},
    {0x1.79c0000000000p-1, 0x1.3763e64645000p-2, 0x1.18b1f291dcb56p-44},
    {0x1.7780000000000p-1, 0x1.3d81fb5947000p-2, -0x1.22c7c2a9d37a4p-45},
    {0x1.7580000000000p-1, 0x1.42f9f3ff62000p-2, 0x1.906440f7d3354p-44},
    {0x1.7340000000000p-1, 0x1.4929e8db4e000p-2, 0x1.b9056556c70dep-44},
    {0x1.7140000000000p-1, 0x1.4eb1f36b07000p-2, 0x1.8404746e5797bp-46},
    {0x1.6f40000000000p-1, 0x1.5441aecbc6000p-2, 0x1.258e66008d39bp-45},
    {0x1.6d00000000000p-1, 0x1.5a8cadbbee000p-2, -0x1.7c79b0af7ecf8p-48},
    {0x1.6b00000000000p-1, 0x1.602d08af09000p-2, 0x1.ebe9176df3f65p-46},
    {0x1.6900000000000p-1, 0x1.65d558d4ce000p-2, 0x1.544fd2dc5bdc0p-51},
    {0x1.6700000000000p-1, 0x1.6b85b4cffa000p-2, 0x1.fe6750d372503p-45},
    {0x1.6540000000000p-1, 0x1.7086b1162b000p-2, 0x1.0fb1677aae284p-44},
    {0x1.6340000000000p-1, 0x1.76466197e3000p-2, 0x1.b7826eb8babdfp-44},
    {0x1.6140000000000p-1, 0x1.7c0e612786000p-2, -0x1.c64e11d8f5a7ep-45},
    {0x1.5f80000000000p-1, 0x1.812444990b000p-2, -0x1.3a3e94cca13d1p-47},
    {0x1.5d80000000000p-1, 0x1.86fc19d051000p-2, 0x1.239fc8edbd99ap-44},
    {0x1.5bc0000000000p-1, 0x1.8c1ffe4002000p-2, 0x1.27c2eca0dbcb6p-45},
    {0x1.59c0000000000p-1, 0x1.920800ccb9000p-2, 0x1.8d62ee5eac0d7p-44},
    {0x1.5800000000000p-1, 0x1.973a343135000p-2, 0x1.ab73b16bf4984p-44},
    {0x1.5640000000000p-1, 0x1.9c73305d48000p-2, -0x1.44e11363841bfp-46},
    {0x1.5480000000000p+0, -0x1.241558bfd1000p-2, -0x1.00fff3228fcadp-44},
    {0x1.52a0000000000p+0, -0x1.1e6dd5557e000p-2, -0x1.eb09e3695e5fdp-44},
    {0x1.5100000000000p+0, -0x1.1980d2dd42000p-2, -0x1.b7b3a7a361c9ap-45},
    {0x1.4f40000000000p+0, -0x1.142bfeb9a0000p-2, -0x1.1ce6185b58a9ep-44},
    {0x1.4d80000000000p+0, -0x1.0ed005f658000p-2, 0x1.2dc75285aa803p-45},
    {0x1.4be0000000000p+0, -0x1.09cf9680ff000p-2, 0x1.7831b71987419p-44},
    {0x1.4a20000000000p+0, -0x1.0465a08155000p-2, 0x1.905f0ad83878ep-52},
    {0x1.4880000000000p+0, -0x1.feb0233e60000p-3, -0x1.f316e32d5e8c7p-45},
    {0x1.46e0000000000p+0, -0x1.f488311d1c000p-3, 0x1.6da82c5068606p-44},
    {0x1.4540000000000p+0, -0x1.ea5349e23a000p-3, -0x1.81b934c73ccb5p-44},
    {0x1.43a0000000000p+0, -0x1.e0114c5332000p-3, 0x1.a0452642f2ab1p-45},
    {0x1.4200000000000p+0, -0x1.d5c216b4fc000p-3, 0x1.1ba91bbca681bp-45},
    {0x1.4080000000000p+0, -0x1.cc320c0176000p-3, -0x1.409039a653794p-45},
    {0x1.3ee0000000000p+0, -0x1.c1c909e2d8000p-3, 0x1.0bd1010c910fap-45},
    {0x1.3d60000000000p+0, -0x1.b820f2fc7e000p-3, -0x1.42177bcc3821ep-45},
    {0x1.3be0000000000p+0, -0x1.ae6d25f274000p-3, -0x1.95d95a1c6908ep-46},
    {0x1.3a60000000000p+0, -0x1.a4ad8639d6000p-3, 0x1.7469948748b19p-44},
    {0x1.38e0000000000p+0, -0x1.9ae1f6dee6000p-3, 0x1.21d7c3601090fp-45},
    {0x1.3760000000000p+0, -0x1.910a5a830e000p-3, -0x1.e75fb5c93ca03p-48},
    {0x1.35e0000000000p+0, -0x1.8726935aca000p-3, -0x1.8c4bb263232fbp-44},
    {0x1.3460000000000p+0, -0x1.7d36832b90000p-3, 0x1.e3a5d33dd3948p-44},
    {0x1.3300000000000p+0, -0x1.740f8f5404000p-3, 0x1.0b66c99018aa1p-44},
    {0x1.3180000000000p+0, -0x1.6a079d0f7a000p-3, -0x1.5a3f8448d14f5p-44},
    {0x1.3020000000000p+0, -0x1.60ca8fe886000p-3, 0x1.d42dd78059eb0p-45},
    {0x1.2ec0000000000p+0, -0x1.5782cb3092000p-3, 0x1.3a46351794442p-44},
    {0x1.2d60000000000p+0, -0x1.4e3035ed50000p-3, 0x1.59adbf9390e52p-44},
    {0x1.2be0000000000p+0, -0x1.43f837179e000p-3, -0x1.52c0a1a8c730ep-44},
    {0x1.2aa0000000000p+0, -0x1.3b6a34236e000p-3, -0x1.5238664434197p-49},
    {0x1.2940000000000p+0, -0x1.31f693eb1a000p-3, 0x1.a6726e5a396fbp-45},
    {0x1.27e0000000000p+0, -0x1.2877bbc0b6000p-3, -0x1.74be8dfa16db8p-44},
    {0x1.2680000000000p+0, -0x1.1eed90e2dc000p-3, -0x1.615637097648fp-46},
    {0x1.2540000000000p+0, -0x1.16377fb124000p-3, -0x1.91e1abf41763ep-47},
    {0x1.23e0000000000p+0, -0x1.0c976b47be000p-3, 0x1.d20254dcd2c22p-45},
    {0x1.22a0000000000p+0, -0x1.03cd40a51a000p-3, -0x1.81a979c146707p-44},
    {0x1.2160000000000p+0, -0x1.f5f2c61e80000p-4, -0x1.df631d467889cp-45},
    {0x1.2020000000000p+0, -0x1.e4377a0da4000p-4, -0x1.36e14aae6add5p-45},
    {0x1.1ec0000000000p+0, -0x1.d09f72b4c4000p-4, -0x1.048c000354e33p-45},
    {0x1.1d80000000000p+0, -0x1.beba818148000p-4, 0x1.89b78b6df1f57p-44},
    {0x1.1c60000000000p+0, -0x1.ae8e7a1050000p-4, 0x1.437ea278af778p-44},
    {0x1.1b20000000000p+0, -0x1.9c83311a54000p-4, 0x1.19742dbf9ee2dp-44},
    {0x1.19e0000000000p+0, -0x1.8a6377a914000p-4, -0x1.c28bb5a46418ap-44},
    {0x1.18a0000000000p+0, -0x1.782f1f39bc000p-4, 0x1.0d5f31f4f972cp-44},
    {0x1.1780000000000p+0, -0x1.67bb0726ec000p-4, -0x1.f724b69ef5912p-49},
    {0x1.1640000000000p+0, -0x1.555efe40b4000p-4, -0x1.0b4978c868e23p-44},
    {0x1.1520000000000p+0, -0x1.44c6dfb9b8000p-4, 0x1.3f34507cbbd76p-45},
    {0x1.1400000000000p+0, -0x1.341d7961bc000p-4, -0x1.1d09299837610p-44},
    {0x1.12c0000000000p+0, -0x1.2185b3b75c000p-4, 0x1.e3189f8f32304p-44},
    {0x1.11a0000000000p+0, -0x1.10b75afd68000p-4, 0x1.f39e8ccf1a6e1p-44},
    {0x1.1080000000000p+0, -0x1.ffae9119b8000p-5, -0x1.303374262c554p-45},
    {0x1.0f60000000000p+0, -0x1.ddcaadb470000p-5, 0x1.0e4f7b2a48432p-45},
    {0x1.0e40000000000p+0, -0x1.bbc2bfc450000p-5, 0x1.7d18691417dafp-46},
    {0x1.0d20000000000p+0, -0x1.99967a4f28000p-5, -0x1.8e432ed72ea8ap-44},
    {0x1.0c00000000000p+0, -0x1.77458f6330000p-5, 0x1.181dce586af09p-44},
    {0x1.0b00000000000p+0, -0x1.58a5bafc90000p-5, 0x1.b2b739570ad39p-45},
    {0x1.09e0000000000p+0, -0x1.360ebf5d80000p-5, -0x1.bb2b2503a5a59p-44},
    {0x1.08c0000000000p+0, -0x1.1352378598000p-5, 0x1.c1ac3b71fa59bp-46},
    {0x1.07c0000000000p+0, -0x1.e8a3ee30d0000p-6, 0x1.1a9fa3de53900p-45},
    {0x1.06a0000000000p+0, -0x1.a29b453fd0000p-6, 0x1.24488f73b23adp-44},
    {0x1.05a0000000000p+0, -0x1.641a176270000p-6, -0x1.adec6522ee537p-47},
    {0x1.04a0000000000p+0, -0x1.255ba259f0000p-6, -0x1.e38e08390cc75p-44},
    {0x1.0380000000000p+0, -0x1.bcf712c740000p-7, -0x1.c25e097bd9771p-46},
    {0x1.0280000000000p+0, -0x1.3e7295d260000p-7, 0x1.609c1ff29a114p-45},
    {0x1.0180000000000p+0, -0x1.7ee11ebd80000p-8, -0x1.749d3c2d23a07p-47},
    {0x1.0000000000000p+0, 0x0.0p+0, 0x0.0p+0},
};

// 2^(j / 32) = hi + lo
struct ExpEntry {
    double hi, lo;
};
constexpr int EXP_N = 32;
__device__ const ExpEntry EXP_TABLE[EXP_N] = {
    {0x1.0000000000000p+0, 0x0.0p+0},
    {0x1.059b0d3158574p+0, 0x1.d73e2a475b465p-55},
    {0x1.0b5586cf9890fp+0, 0x1.8a62e4adc610bp-54},
    {0x1.11301d0125b51p+0, -0x1.6c51039449b3ap-54},
    {0x1.172b83c7d517bp+0, -0x1.19041b9d78a76p-55},
    {0x1.1d4873168b9aap+0, 0x1.e016e00a2643cp-54},
    {0x1.2387a6e756238p+0, 0x1.9b07eb6c70573p-54},
    {0x1.29e9df51fdee1p+0, 0x1.612e8afad1255p-55},
    {0x1.306fe0a31b715p+0, 0x1.6f46ad23182e4p-55},
    {0x1.371a7373aa9cbp+0, -0x1.63aeabf42eae2p-54},
    {0x1.3dea64c123422p+0, 0x1.ada0911f09ebcp-55},
    {0x1.44e086061892dp+0, 0x1.89b7a04ef80d0p-59},
    {0x1.4bfdad5362a27p+0, 0x1.d4397afec42e2p-56},
    {0x1.5342b569d4f82p+0, -0x1.07abe1db13cadp-55},
    {0x1.5ab07dd485429p+0, 0x1.6324c054647adp-54},
    {0x1.6247eb03a5585p+0, -0x1.383c17e40b497p-54},
    {0x1.6a09e667f3bcdp+0, -0x1.bdd3413b26456p-54},
    {0x1.71f75e8ec5f74p+0, -0x1.16e4786887a99p-55},
    {0x1.7a11473eb0187p+0, -0x1.41577ee04992fp-55},
    {0x1.82589994cce13p+0, -0x1.d4c1dd41532d8p-54},
    {0x1.8ace5422aa0dbp+0, 0x1.6e9f156864b27p-54},
    {0x1.93737b0cdc5e5p+0, -0x1.75fc781b57ebcp-57},
    {0x1.9c49182a3f090p+0, 0x1.c7c46b071f2bep-56},
    {0x1.a5503b23e255dp+0, -0x1.d2f6edb8d41e1p-54},
    {0x1.ae89f995ad3adp+0, 0x1.7a1cd345dcc81p-54},
    {0x1.b7f76f2fb5e47p+0, -0x1.5584f7e54ac3bp-56},
    {0x1.c199bdd85529cp+0, 0x1.11065895048ddp-55},
    {0x1.cb720dcef9069p+0, 0x1.503cbd1e949dbp-56},
    {0x1.d5818dcfba487p+0, 0x1.2ed02d75b3707p-55},
    {0x1.dfc97337b9b5fp+0, -0x1.1a5cd4f184b5cp-54},
    {0x1.ea4afa2a490dap+0, -0x1.e9c23179c2893p-54},
    {0x1.f50765b6e4540p+0, 0x1.9d3e12dd8a18bp-54},
};

// The tables in LDS; stage_math64 is called by every thread of the workgroup,
// followed by a barrier of the caller.
struct Math64 {
    LogEntry log[LOG_N];
    ExpEntry exp[EXP_N];
};

__device__ __forceinline__ void stage_math64(Math64& m)
{
    for (int q = threadIdx.x; q < LOG_N; q += blockDim.x) m.log[q] = LOG_TABLE[q];
    for (int q = threadIdx.x; q < EXP_N; q += blockDim.x) m.exp[q] = EXP_TABLE[q];
}

// sqrt(h) for h = 0, +inf or normal: one Goldschmidt step from the hardware's
// reciprocal square root, then a residual correction.
__device__ __forceinline__ double sqrt_mid(double h)
{
#pragma clang fp contract(off)
    const double y = __builtin_amdgcn_rsq(h);
    double g = h * y, q = 0.5 * y;
    const double e = fma(-q, g, 0.5);
    g = fma(g, e, g);
    q = fma(q, e, q);
    g = fma(fma(-g, g, h), q, g);
    return __builtin_amdgcn_class(h, 0x260) ? h : g;  // +-0, +inf
}

// a / y for normal y and quotient: one Newton step on the hardware's
// reciprocal, then a residual correction.
__device__ __forceinline__ double div_mid(double a, double y)
{
#pragma clang fp contract(off)
    double r = __builtin_amdgcn_rcp(y);
    r = fma(fma(-y, r, 1.0), r, r);
    const double q = a * r;
    return fma(fma(-q, y, a), r, q);
}

// x / P given rP = 1 / P rounded
__device__ __forceinline__ double div_by(double x, double P, double rP)
{
#pragma clang fp contract(off)
    const double q = x * rP;
    return fma(fma(-q, P, x), rP, q);
}

// ln x = hi + lo for positive normal x, hi the rounded value up to 1 ulp. The
// polynomial is summed in pairs (Estrin): the chain is what a walk waits for.
__device__ __forceinline__ double log_parts(double x, const Math64& tab, double& lo)
{
#pragma clang fp contract(off)
    const int hx = __double2hiint(x);
    const int up = hx + (1 << 19);                   // significands from 3/2 on carry into the exponent
    const int e = (up >> 20) - 1023;
    const double z = __hiloint2double(hx - (up & 0x7ff00000) + 0x3ff00000, __double2loint(x));
    const LogEntry t = tab.log[(hx >> 13) & (LOG_N - 1)];
    const double ef = (double)e;
    const double hi = fma(ef, 0x1.62e42fefa3800p-1, t.hi);  // exact
    const double r = fma(z, t.c, -1.0);                     // |r| <= 2^-7
    const double s = hi + r;
    const double w = (hi - s) + r;                          // exact: hi = 0 or |hi| > |r|
    const double r2 = r * r;
    const double p01 = fma(r, 1.0 / 3, -1.0 / 2), p23 = fma(r, 1.0 / 5, -1.0 / 4), p45 = fma(r, 1.0 / 7, -1.0 / 6);
    const double p = fma(r2, fma(r2, fma(r2, -1.0 / 8, p45), p23), p01);
    lo = fma(r2, p, w + fma(ef, 0x1.ef35793c76730p-45, t.lo));
    return s;
}

__device__ __forceinline__ double log_mid(double x, const Math64& tab)
{
#pragma clang fp contract(off)
    double lo;
    const double hi = log_parts(x, tab, lo);
    return hi + lo;
}

// sin and cos of phi in [0, 2 pi]: the nearest multiple of pi / 2 is taken off
// (the first product is exact after cancellation), then one polynomial each.
__device__ __forceinline__ void sincos_turn(double phi, double& sn, double& cs)
{
#pragma clang fp contract(off)
    const double k = rint(phi * 0x1.45f306dc9c883p-1);
    const double r0 = fma(-k, 0x1.921fb54442d18p+0, phi);  // exact
    const double r = fma(-k, 0x1.1a62633145c07p-54, r0);
    const double rl = fma(-k, 0x1.1a62633145c07p-54, r0 - r);  // what r's rounding lost
    const double z = r * r, w = fma(-0.5, z, 1.0);
    double p = fma(z, -0x1.ab17a792c9454p-41, 0x1.61217ec01840fp-33);
    p = fma(z, p, -0x1.ae6454126638cp-26);
    p = fma(z, p, 0x1.71de3a54605eep-19);
    p = fma(z, p, -0x1.a01a01a019936p-13);
    p = fma(z, p, 0x1.1111111111110p-7);
    p = fma(z, p, -0x1.5555555555555p-3);
    const double a = r + fma(r * z, p, rl * w);
    double q = fma(z, -0x1.907d7aec5a8a3p-37, 0x1.1eeb68b109cf5p-29);
    q = fma(z, q, -0x1.27e4fa17a41bfp-22);
    q = fma(z, q, 0x1.a01a019f4e867p-16);
    q = fma(z, q, -0x1.6c16c16c16966p-10);
    q = fma(z, q, 0x1.5555555555555p-5);
    const double b = w + fma(z * z, q, fma(-r, rl, fma(-0.5, z, 1.0 - w)));
    const int n = (int)k;
    const double u = (n & 1) ? b : a, v = (n & 1) ? a : b;
    sn = (n & 2) ? -u : u;
    cs = ((n + 1) & 2) ? -v : v;
}

// M^n for a count M in [1, 2^31) and n in [0, POW_N_MAX] with at most 24
// significant bits: exp(n ln M) with ln M in two parts, the first of 29 bits so
// that its product with n is exact. In two halves, which a walk runs in
// different days: n ln M = hi + lo, and its exponential.
constexpr float POW_N_MAX = 16.0f;
struct PowArg {
    double hi, lo;
};
__device__ __forceinline__ PowArg pow_arg(double M, double n, const Math64& tab)
{
#pragma clang fp contract(off)
    double lo;
    const double s = log_parts(M, tab, lo);
    const double h = __longlong_as_double(__double_as_longlong(s) & ~((1ll << 24) - 1));
    return PowArg{n * h, n * ((s - h) + lo)};
}

__device__ __forceinline__ double pow_exp(PowArg p, const Math64& tab)
{
#pragma clang fp contract(off)
    // k = the nearest integer to hi 32 / ln 2, in the low bits of a sum with 1.5 2^52
    const double kb = fma(p.hi, 0x1.71547652b82fep+5, 0x1.8p+52);
    const int ki = __double2loint(kb);
    const double k = kb - 0x1.8p+52;
    double r = fma(-k, 0x1.62e42fefa0000p-6, p.hi);
    r = fma(-k, 0x1.cf79abc9e3b3ap-45, r) + p.lo;  // |r| < 0.011
    const ExpEntry t = tab.exp[ki & (EXP_N - 1)];
    const double r2 = r * r;
    const double q = fma(r2, fma(r2, fma(r, 1.0 / 720, 1.0 / 120), fma(r, 1.0 / 24, 1.0 / 6)) * r, fma(0.5, r2, r));
    return __builtin_amdgcn_ldexp(t.hi + fma(t.hi, q, t.lo), ki >> 5);
}

}  // namespace abc
