// Fused vocab-wide softmax statistics, speculative accept, residual resample and
// behavior log-probs (the serving engine's speculative-decoding accept rule with
// temperature 1 and no truncation; paper Sec. 4.1 control table, Sec. 4.2, Sec. 5.3/5.4;
// rule of Leviathan et al. 2023 / Chen et al. 2023).
//
// Four launches (with few sequences three, 2 inside 3), all deterministic (fixed reduction orders, integer prefix sums, no
// atomics):
//   1. chunk_stats  grid = rows * chunks: per 8192-logit chunk its max and
//                   sum exp(l - chunk max) (f32 exp2 with the roundings of the difference and
//                   of the base change compensated, f64 accumulation across threads).
//   2. decide       one workgroup per sequence: row moments (m, S) from the chunk
//                   statistics, the k tests u*q*S < exp(l_x - m) in f64, the accepted drafts
//                   with their log-probs, n, and the descriptor of the final draw.
//   3. mass         grid = 4 B * chunks: the integer mass floor(r_t 2^62) of each logit of the
//                   final draw's row (residual max(0, p - q), or p for a bonus draw; p_t to
//                   ~1e-10 relative, so that the only rounding that matters in the draw is
//                   that of S, which scales every mass alike), summed per 256-logit
//                   sub-block.
//   4. draw_pick    one wavefront per sequence: Tot, target = (Tot * floor(u 2^32)) >> 32,
//                   then three integer prefix searches (chunk, sub-block, 4 logits per lane)
//                   that recompute only the one sub-block's masses.
// Bytes: pass 1 reads the B(1+k)V logits once; pass 3 reads one row (+ one q row on a
// rejection) per sequence; pass 4 reads 1 KB (+ 1 KB) per sequence. Pass 1 and 3 are VALU
// bound as much as HBM bound (without packed math a wave64 instruction takes 4 cycles), so
// their per-logit instruction counts are kept small.
#include <type_traits>

#include "device_common.h"
#include "internal.h"

// The draw recomputes masses in two kernels; both must round identically, so no
// floating-point contraction in this file.
#pragma clang fp contract(off)

namespace molt {
namespace {

constexpr int kThreads = 256;
constexpr int kPerThread = 32;
constexpr int kChunk = kThreads * kPerThread;  // 8192 logits per chunk
constexpr int kSub = 4 * kWave;                // 256 logits per draw sub-block
constexpr int kSubs = kChunk / kSub;           // 32 sub-blocks per chunk
constexpr int kRowsPerBatch = 16;              // accept rows examined per batch (4 per wave)
constexpr float kL2e = 0x1.715476p+0f;         // log2(e) rounded to f32
constexpr float kL2eLo = 0x1.4ae0c0p-26f;      // log2(e) - kL2e
constexpr float kLn2 = 0x1.62e430p-1f;         // ln 2
constexpr float kSparse = 0x1p30f;             // logits this large: spacing 64 below, 128 above

struct FinalDraw {
  double m;      // row max
  double S;      // row sum exp(l - m)
  int row;       // row index inside the sequence (0..k)
  int mode;      // 0: draw from p, 1: residual with q row, 2: residual with one-hot q
  int draft;     // the rejected draft (mode 2)
  int pad;
};

// ---- pass 1 ---------------------------------------------------------------------------
template <bool kVec>
__global__ __launch_bounds__(kThreads) void chunk_stats_kernel(const float* __restrict__ logits,
                                                               long rows, int V, int nch,
                                                               float* __restrict__ cmax,
                                                               double* __restrict__ csum) {
  __shared__ float redf[kThreads / kWave];
  __shared__ double redd[kThreads / kWave];
  const long id = blockIdx.x;
  const long row = id / nch;
  const int c = int(id % nch);
  const float* src = logits + row * long(V) + long(c) * kChunk;
  const int n = min(kChunk, V - c * kChunk);
  float v[kPerThread];
  if (kVec) {
    // 16-byte nontemporal loads (each logit is read once here), element 4*(tid + 256 i) + e,
    // from clamped addresses so that no branch separates them (n % 4 == 0 here)
#pragma unroll
    for (int i = 0; i < kPerThread / 4; ++i) {
      const int e0 = 4 * (threadIdx.x + kThreads * i);
      const floatx4_t t = __builtin_nontemporal_load(reinterpret_cast<const floatx4_t*>(src + min(e0, n - 4)));
      const bool in = e0 < n;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * i + e] = in ? t[e] : -INFINITY;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      int e = threadIdx.x + kThreads * i;
      v[i] = e < n ? src[e] : -INFINITY;
    }
  }
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) mx = fmaxf(mx, v[i]);
  mx = block_max<kThreads / kWave>(mx, redf);
  float s = 0.f;
  if (fabsf(mx) >= kSparse && mx != INFINITY && mx != -INFINITY) {
    // f32 logits of this size lie 64 and more apart: all but those equal to mx weigh under 2^-92
    // (and mx - 200 below may round to mx)
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) s += v[i] == mx ? 1.f : 0.f;
  } else if (mx != -INFINITY) {
    // exp(l - mx) to ~1 ulp with every rounding compensated: logits below mx - 200 (and the
    // padding's -inf) are raised to it, where exp underflows to 0 in f32; d + err == l - mx
    // exactly (TwoSum); d log2(e) = t + terr (FMA split, log2(e) = kL2e + kL2eLo); then
    // exp(l - mx) = 2^t * exp(terr ln2 + err) ~ 2^t (1 + terr ln2 + err), with 2^t from the
    // hardware exp2 (1 ulp)
    const float lo = mx - 200.0f, nmx = -mx;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const float vc = fmaxf(v[i], lo);
      const float d = vc + nmx;
      const float bb = d - vc;
      const float err = (vc - (d - bb)) + (nmx - bb);
      const float t = d * kL2e;
      const float terr = fmaf(d, kL2eLo, fmaf(d, kL2e, -t));
      const float e = __builtin_amdgcn_exp2f(t);
      s += fmaf(e, fmaf(terr, kLn2, err), e);
    }
  }
  double sd = block_sum<kThreads / kWave, double>(double(s), redd);
  if (threadIdx.x == 0) {
    cmax[id] = mx;
    csum[id] = sd;
  }
}

// inclusive prefix sum over the wavefront (integers: exact)
MOLT_DEV unsigned long long wave_incl_scan(unsigned long long v, int lane) {
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const unsigned long long u = __shfl_up(v, o, kWave);
    if (lane >= o) v += u;
  }
  return v;
}

// exp(x) for x <= 0 by the table-driven method of P. T. P. Tang (ACM TOMS 15(2), 1989):
// x = (256 m + j) ln2/256 + r with |r| <= ln2/512 (reduction in f64, exact), exp(x) =
// 2^m * 2^(j/256) * (1 + p(r)), tab[j] = 2^(j/256) in f64 (copied to LDS by exp_table_init)
// and p(r) = r + r^2/2 + r^3/6 evaluated in f32: |p| < 1.4e-3, so its f32 rounding and the
// truncation (r^4/24 < 1.4e-13) leave a relative error below 3e-10, far inside the 2e-8 of
// the integer total within which a draw counts as a near-tie. About a third of the
// instructions of a library f64 exp; the draw evaluates it for every logit of B rows.
// The power of two goes into the exponent bits of the table value, which a caller may have scaled
// (by 1 / S); n is rounded by adding 1.5 * 2^52, whose sum carries it in its low word. x has to be
// at least kExpMin, so that exponents stay in range.
constexpr double kExpInvL = 0x1.71547652b82fep+8;   // 256 / ln2
constexpr double kExpLhi = 0x1.62e42fef80000p-9;    // ln2 / 256, 34 significant bits
constexpr double kExpLlo = 0x1.1cf79abc9e3b4p-44;   // ln2 / 256 - kExpLhi
constexpr double kExpRound = 0x1.8p+52;
constexpr double kExpMin = -600.0;

MOLT_DEV double exp_nonpos(double x, const double* tab) {
  const double nr = fma(x, kExpInvL, kExpRound);
  const int N = __double2loint(nr);
  const double n = nr - kExpRound;
  double r = fma(-n, kExpLhi, x);                    // exact: n * kExpLhi has <= 53 bits
  r = fma(-n, kExpLlo, r);
  const float rf = float(r);
  const float pf = rf * fmaf(rf, fmaf(rf, 1.0f / 6.0f, 0.5f), 1.0f);
  const double t = tab[N & 255];
  const double y = fma(t, double(pf), t);
  return __hiloint2double(__double2hiint(y) + ((N >> 8) << 20), __double2loint(y));   // N >> 8 == floor(N / 256)
}

// 2^(j / 256), j < 256, correctly rounded
__device__ const double kExpTable[256] = {
    0x1.0000000000000p+0, 0x1.00b1afa5abcbfp+0, 0x1.0163da9fb3335p+0, 0x1.02168143b0281p+0,
    0x1.02c9a3e778061p+0, 0x1.037d42e11bbccp+0, 0x1.04315e86e7f85p+0, 0x1.04e5f72f654b1p+0,
    0x1.059b0d3158574p+0, 0x1.0650a0e3c1f89p+0, 0x1.0706b29ddf6dep+0, 0x1.07bd42b72a836p+0,
    0x1.0874518759bc8p+0, 0x1.092bdf66607e0p+0, 0x1.09e3ecac6f383p+0, 0x1.0a9c79b1f3919p+0,
    0x1.0b5586cf9890fp+0, 0x1.0c0f145e46c85p+0, 0x1.0cc922b7247f7p+0, 0x1.0d83b23395decp+0,
    0x1.0e3ec32d3d1a2p+0, 0x1.0efa55fdfa9c5p+0, 0x1.0fb66affed31bp+0, 0x1.1073028d7233ep+0,
    0x1.11301d0125b51p+0, 0x1.11edbab5e2ab6p+0, 0x1.12abdc06c31ccp+0, 0x1.136a814f204abp+0,
    0x1.1429aaea92de0p+0, 0x1.14e95934f312ep+0, 0x1.15a98c8a58e51p+0, 0x1.166a45471c3c2p+0,
    0x1.172b83c7d517bp+0, 0x1.17ed48695bbc0p+0, 0x1.18af9388c8deap+0, 0x1.1972658375d2fp+0,
    0x1.1a35beb6fcb75p+0, 0x1.1af99f8138a1cp+0, 0x1.1bbe084045cd4p+0, 0x1.1c82f95281c6bp+0,
    0x1.1d4873168b9aap+0, 0x1.1e0e75eb44027p+0, 0x1.1ed5022fcd91dp+0, 0x1.1f9c18438ce4dp+0,
    0x1.2063b88628cd6p+0, 0x1.212be3578a819p+0, 0x1.21f49917ddc96p+0, 0x1.22bdda27912d1p+0,
    0x1.2387a6e756238p+0, 0x1.2451ffb82140ap+0, 0x1.251ce4fb2a63fp+0, 0x1.25e85711ece75p+0,
    0x1.26b4565e27cddp+0, 0x1.2780e341ddf29p+0, 0x1.284dfe1f56381p+0, 0x1.291ba7591bb70p+0,
    0x1.29e9df51fdee1p+0, 0x1.2ab8a66d10f13p+0, 0x1.2b87fd0dad990p+0, 0x1.2c57e39771b2fp+0,
    0x1.2d285a6e4030bp+0, 0x1.2df961f641589p+0, 0x1.2ecafa93e2f56p+0, 0x1.2f9d24abd886bp+0,
    0x1.306fe0a31b715p+0, 0x1.31432edeeb2fdp+0, 0x1.32170fc4cd831p+0, 0x1.32eb83ba8ea32p+0,
    0x1.33c08b26416ffp+0, 0x1.3496266e3fa2dp+0, 0x1.356c55f929ff1p+0, 0x1.36431a2de883bp+0,
    0x1.371a7373aa9cbp+0, 0x1.37f26231e754ap+0, 0x1.38cae6d05d866p+0, 0x1.39a401b7140efp+0,
    0x1.3a7db34e59ff7p+0, 0x1.3b57fbfec6cf4p+0, 0x1.3c32dc313a8e5p+0, 0x1.3d0e544ede173p+0,
    0x1.3dea64c123422p+0, 0x1.3ec70df1c5175p+0, 0x1.3fa4504ac801cp+0, 0x1.40822c367a024p+0,
    0x1.4160a21f72e2ap+0, 0x1.423fb2709468ap+0, 0x1.431f5d950a897p+0, 0x1.43ffa3f84b9d4p+0,
    0x1.44e086061892dp+0, 0x1.45c2042a7d232p+0, 0x1.46a41ed1d0057p+0, 0x1.4786d668b3237p+0,
    0x1.486a2b5c13cd0p+0, 0x1.494e1e192aed2p+0, 0x1.4a32af0d7d3dep+0, 0x1.4b17dea6db7d7p+0,
    0x1.4bfdad5362a27p+0, 0x1.4ce41b817c114p+0, 0x1.4dcb299fddd0dp+0, 0x1.4eb2d81d8abffp+0,
    0x1.4f9b2769d2ca7p+0, 0x1.508417f4531eep+0, 0x1.516daa2cf6642p+0, 0x1.5257de83f4eefp+0,
    0x1.5342b569d4f82p+0, 0x1.542e2f4f6ad27p+0, 0x1.551a4ca5d920fp+0, 0x1.56070dde910d2p+0,
    0x1.56f4736b527dap+0, 0x1.57e27dbe2c4cfp+0, 0x1.58d12d497c7fdp+0, 0x1.59c0827ff07ccp+0,
    0x1.5ab07dd485429p+0, 0x1.5ba11fba87a03p+0, 0x1.5c9268a5946b7p+0, 0x1.5d84590998b93p+0,
    0x1.5e76f15ad2148p+0, 0x1.5f6a320dceb71p+0, 0x1.605e1b976dc09p+0, 0x1.6152ae6cdf6f4p+0,
    0x1.6247eb03a5585p+0, 0x1.633dd1d1929fdp+0, 0x1.6434634ccc320p+0, 0x1.652b9febc8fb7p+0,
    0x1.6623882552225p+0, 0x1.671c1c70833f6p+0, 0x1.68155d44ca973p+0, 0x1.690f4b19e9538p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6b052fa75173ep+0, 0x1.6c012750bdabfp+0, 0x1.6cfdcddd47645p+0,
    0x1.6dfb23c651a2fp+0, 0x1.6ef9298593ae5p+0, 0x1.6ff7df9519484p+0, 0x1.70f7466f42e87p+0,
    0x1.71f75e8ec5f74p+0, 0x1.72f8286ead08ap+0, 0x1.73f9a48a58174p+0, 0x1.74fbd35d7cbfdp+0,
    0x1.75feb564267c9p+0, 0x1.77024b1ab6e09p+0, 0x1.780694fde5d3fp+0, 0x1.790b938ac1cf6p+0,
    0x1.7a11473eb0187p+0, 0x1.7b17b0976cfdbp+0, 0x1.7c1ed0130c132p+0, 0x1.7d26a62ff86f0p+0,
    0x1.7e2f336cf4e62p+0, 0x1.7f3878491c491p+0, 0x1.80427543e1a12p+0, 0x1.814d2add106d9p+0,
    0x1.82589994cce13p+0, 0x1.8364c1eb941f7p+0, 0x1.8471a4623c7adp+0, 0x1.857f4179f5b21p+0,
    0x1.868d99b4492edp+0, 0x1.879cad931a436p+0, 0x1.88ac7d98a6699p+0, 0x1.89bd0a478580fp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8be05bad61778p+0, 0x1.8cf3216b5448cp+0, 0x1.8e06a5e0866d9p+0,
    0x1.8f1ae99157736p+0, 0x1.902fed0282c8ap+0, 0x1.9145b0b91ffc6p+0, 0x1.925c353aa2fe2p+0,
    0x1.93737b0cdc5e5p+0, 0x1.948b82b5f98e5p+0, 0x1.95a44cbc8520fp+0, 0x1.96bdd9a7670b3p+0,
    0x1.97d829fde4e50p+0, 0x1.98f33e47a22a2p+0, 0x1.9a0f170ca07bap+0, 0x1.9b2bb4d53fe0dp+0,
    0x1.9c49182a3f090p+0, 0x1.9d674194bb8d5p+0, 0x1.9e86319e32323p+0, 0x1.9fa5e8d07f29ep+0,
    0x1.a0c667b5de565p+0, 0x1.a1e7aed8eb8bbp+0, 0x1.a309bec4a2d33p+0, 0x1.a42c980460ad8p+0,
    0x1.a5503b23e255dp+0, 0x1.a674a8af46052p+0, 0x1.a799e1330b358p+0, 0x1.a8bfe53c12e59p+0,
    0x1.a9e6b5579fdbfp+0, 0x1.ab0e521356ebap+0, 0x1.ac36bbfd3f37ap+0, 0x1.ad5ff3a3c2774p+0,
    0x1.ae89f995ad3adp+0, 0x1.afb4ce622f2ffp+0, 0x1.b0e07298db666p+0, 0x1.b20ce6c9a8952p+0,
    0x1.b33a2b84f15fbp+0, 0x1.b468415b749b1p+0, 0x1.b59728de5593ap+0, 0x1.b6c6e29f1c52ap+0,
    0x1.b7f76f2fb5e47p+0, 0x1.b928cf22749e4p+0, 0x1.ba5b030a1064ap+0, 0x1.bb8e0b79a6f1fp+0,
    0x1.bcc1e904bc1d2p+0, 0x1.bdf69c3f3a207p+0, 0x1.bf2c25bd71e09p+0, 0x1.c06286141b33dp+0,
    0x1.c199bdd85529cp+0, 0x1.c2d1cd9fa652cp+0, 0x1.c40ab5fffd07ap+0, 0x1.c544778fafb22p+0,
    0x1.c67f12e57d14bp+0, 0x1.c7ba88988c933p+0, 0x1.c8f6d9406e7b5p+0, 0x1.ca3405751c4dbp+0,
    0x1.cb720dcef9069p+0, 0x1.ccb0f2e6d1675p+0, 0x1.cdf0b555dc3fap+0, 0x1.cf3155b5bab74p+0,
    0x1.d072d4a07897cp+0, 0x1.d1b532b08c968p+0, 0x1.d2f87080d89f2p+0, 0x1.d43c8eacaa1d6p+0,
    0x1.d5818dcfba487p+0, 0x1.d6c76e862e6d3p+0, 0x1.d80e316c98398p+0, 0x1.d955d71ff6075p+0,
    0x1.da9e603db3285p+0, 0x1.dbe7cd63a8315p+0, 0x1.dd321f301b460p+0, 0x1.de7d5641c0658p+0,
    0x1.dfc97337b9b5fp+0, 0x1.e11676b197d17p+0, 0x1.e264614f5a129p+0, 0x1.e3b333b16ee12p+0,
    0x1.e502ee78b3ff6p+0, 0x1.e653924676d76p+0, 0x1.e7a51fbc74c83p+0, 0x1.e8f7977cdb740p+0,
    0x1.ea4afa2a490dap+0, 0x1.eb9f4867cca6ep+0, 0x1.ecf482d8e67f1p+0, 0x1.ee4aaa2188510p+0,
    0x1.efa1bee615a27p+0, 0x1.f0f9c1cb6412ap+0, 0x1.f252b376bba97p+0, 0x1.f3ac948dd7274p+0,
    0x1.f50765b6e4540p+0, 0x1.f6632798844f8p+0, 0x1.f7bfdad9cbe14p+0, 0x1.f91d802243c89p+0,
    0x1.fa7c1819e90d8p+0, 0x1.fbdba3692d514p+0, 0x1.fd3c22b8f71f1p+0, 0x1.fe9d96b2a23d9p+0};

// tab[j] = scale * 2^(j / 256), j < 256, by nthreads threads; the caller synchronises
MOLT_DEV void exp_table_init(double* tab, double scale, int tid, int nthreads) {
  for (int j = tid; j < 256; j += nthreads) tab[j] = scale * kExpTable[j];
}

// floor(r * 2^62) for 0 < r <= 1 + 2^-52, from the bits of r = mant * 2^(e - 52)
MOLT_DEV unsigned long long grid_floor(double r) {
  const uint32_t hi = uint32_t(__double2hiint(r));
  const unsigned long long mant =
      (static_cast<unsigned long long>((hi & 0xfffffu) | 0x100000u) << 32) | uint32_t(__double2loint(r));
  const int down = 1023 - int(hi >> 20);             // -e >= 0
  return (mant << 10) >> min(down, 63);              // mant << 10 < 2^63
}

// Logits below m - 64 have p < 2^-62, mass 0 whatever q is: their difference (-inf and NaN too) is
// raised to kMassMin, which keeps exp_nonpos in its range. The difference in f64 and not the logit in
// f32, where m - 64 is m itself from |m| = 2^30 on and every logit would be raised to the largest.
constexpr double kMassMin = -64.0;

// residual mass of one logit on the 2^62 grid; tab is scaled by 1 / S, so that the exponential is
// p_t (only S's rounding remains)
MOLT_DEV unsigned long long grid_mass(float l, double m, int mode, float qv, bool is_draft,
                                      const double* tab) {
  const double p = exp_nonpos(fmax(double(l) - m, kMassMin), tab);
  double r = p;
  if (mode == 1) r = p - double(qv);
  else if (mode == 2 && is_draft) r = p - 1.0;
  return r > 0.0 ? grid_floor(r) : 0ull;
}

// The 4 consecutive logits [t0, t0 + 4) of a draw row and, for a residual draw against a
// q row, their q values (0 past V). Loads are issued separately from the arithmetic so that
// a thread's loads are all in flight before the first exp waits on one.
struct Quad {
  float l[4], q[4];
};

template <bool kVec>
MOLT_DEV void quad_load(const float* lrow, const float* qrow, int t0, int V, int mode, Quad& d) {
  // Unconditional loads from clamped addresses (values past V are masked by quad_mass; a
  // non-residual draw reads its logits row again in place of q): no branch separates a
  // load from the next one, so none waits for an earlier one to return.
  const float* qsrc = mode == 1 ? qrow : lrow;
  if (kVec) {
    const int a = min(t0, V - 4);       // V % 4 == 0, V >= 4: the quad is all in or all out
    const float4 x = *reinterpret_cast<const float4*>(lrow + a);
    const float4 y = *reinterpret_cast<const float4*>(qsrc + a);
    d.l[0] = x.x; d.l[1] = x.y; d.l[2] = x.z; d.l[3] = x.w;
    d.q[0] = y.x; d.q[1] = y.y; d.q[2] = y.z; d.q[3] = y.w;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int a = min(t0 + e, V - 1);
      d.l[e] = lrow[a];
      d.q[e] = qsrc[a];
    }
  }
}

// masses of a loaded quad (0 past V, and where the row's sum is not a number), and their sum
MOLT_DEV unsigned long long quad_mass(const Quad& d, int t0, int V, const FinalDraw& f, int mode,
                                      const double* tab, unsigned long long (&g)[4]) {
  unsigned long long sum = 0;
  const int n = f.S > 0.0 ? V : 0;
  const int dr = f.draft - t0;                       // the draft's place in the quad, if any
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    g[e] = t0 + e < n ? grid_mass(d.l[e], f.m, mode, d.q[e], dr == e, tab) : 0ull;
    sum += g[e];
  }
  return sum;
}

// ---- pass 2 ---------------------------------------------------------------------------
// One workgroup per sequence: its accept decisions, batches of 16 rows (row r on wavefront
// r % 4): row moments (m, S) from the chunk statistics, the tests u*q*S < exp(l_x - m) in
// f64, n, and the descriptor of the final draw, which is returned. With `write` the accepted
// drafts (where out_tokens is given), their log-probs, n and the descriptor are stored too.
MOLT_DEV FinalDraw decide(const float* __restrict__ logits, const float* __restrict__ q,
                          const int32_t* __restrict__ drafts, const float* __restrict__ u, int b,
                          int k, int V, int nch, const float* __restrict__ cmax,
                          const double* __restrict__ csum, int dstride, int doff, bool write,
                          int32_t* __restrict__ out_tokens, int32_t* __restrict__ out_n,
                          float* __restrict__ out_lp, FinalDraw* __restrict__ fin) {
  __shared__ double s_m[kRowsPerBatch], s_S[kRowsPerBatch], s_lx[kRowsPerBatch];
  __shared__ int s_ok[kRowsPerBatch], s_x[kRowsPerBatch];
  __shared__ int s_n;
  __shared__ FinalDraw s_fin;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const long r0 = long(b) * (k + 1);
  if (threadIdx.x == 0) s_n = -1;
  // ---- the sequence's decisions, batches of 16 rows (row r on wavefront r % 4)
  for (int base = 0; base <= k; base += kRowsPerBatch) {
    constexpr int kPer = kRowsPerBatch / 4;
    float cm[kPer];
    double cs[kPer];
    int xv[kPer];
    float uv[kPer];
    // issue every load of the batch first: chunk statistics (lane = chunk) and, on lane 0,
    // the draft id and its uniform
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int r = base + wave + 4 * j;
      cm[j] = -INFINITY;
      cs[j] = 0.0;
      xv[j] = -1;
      uv[j] = 0.f;
      if (r <= k && lane < nch) {
        cm[j] = cmax[(r0 + r) * nch + lane];
        cs[j] = csum[(r0 + r) * nch + lane];
      }
      if (r < k && lane == 0) {
        xv[j] = drafts[long(b) * dstride + doff + r];
        uv[j] = u[r0 + r];
      }
    }
    float lxv[kPer];
    float qxv[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int r = base + wave + 4 * j;
      lxv[j] = 0.f;
      qxv[j] = 1.f;
      const int x = xv[j];
      if (r < k && lane == 0 && x >= 0 && x < V) {
        lxv[j] = logits[(r0 + r) * V + x];
        if (q) qxv[j] = q[(long(b) * k + r) * V + x];
      }
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int r = base + wave + 4 * j;
      if (r > k) break;
      // row moments: m = max of the chunk maxima, S = sum csum * exp(cmax - m) (f64)
      float mx = -INFINITY;
      for (int cc = lane; cc < nch; cc += kWave) {
        const float v = cc == lane ? cm[j] : cmax[(r0 + r) * nch + cc];
        mx = fmaxf(mx, v);
      }
      mx = wave_max(mx);
      double acc = 0.0;
      for (int cc = lane; cc < nch; cc += kWave) {
        const float v = cc == lane ? cm[j] : cmax[(r0 + r) * nch + cc];
        const double sv = cc == lane ? cs[j] : csum[(r0 + r) * nch + cc];
        if (v != -INFINITY) acc += sv * exp(double(v) - double(mx));
      }
      acc = wave_sum(acc);
      if (lane == 0) {
        const int i = r - base;
        const double m = double(mx);
        s_m[i] = m;
        s_S[i] = acc;
        s_x[i] = xv[j];
        s_ok[i] = 0;
        if (r < k) {
          const int x = xv[j];
          bool accept = false;
          double lx = 0.0;
          if (x >= 0 && x < V) {
            lx = double(lxv[j]);
            const double ex = exp(lx - m);
            const double qx = q ? double(qxv[j]) : 1.0;
            accept = double(uv[j]) * qx * acc < ex;
          }
          s_ok[i] = accept;
          s_lx[i] = lx;
        }
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      // first rejection in this batch decides n; accepted rows before it are emitted
      const int last = min(k, base + kRowsPerBatch - 1);
      for (int r = base; r <= last; ++r) {
        const int i = r - base;
        if (r == k || !s_ok[i]) {
          s_n = r;
          FinalDraw f;
          f.m = s_m[i];
          f.S = s_S[i];
          f.row = r;
          f.mode = r == k ? 0 : (q ? 1 : 2);
          f.draft = r == k ? -1 : s_x[i];
          f.pad = 0;
          s_fin = f;
          break;
        }
        if (!write) continue;
        if (out_tokens) out_tokens[r0 + r] = s_x[i];
        if (out_lp) out_lp[r0 + r] = float((s_lx[i] - s_m[i]) - log(s_S[i]));
      }
    }
    __syncthreads();
    if (s_n >= 0) break;
  }
  if (!write) return s_fin;
  const int n = s_n;
  for (int j = n + 1 + int(threadIdx.x); j <= k; j += kThreads) {
    if (out_tokens) out_tokens[r0 + j] = -1;
    if (out_lp) out_lp[r0 + j] = __builtin_nanf("");
  }
  if (threadIdx.x == 0) {
    out_n[b] = n;
    fin[b] = s_fin;
  }
  return s_fin;
}

__global__ __launch_bounds__(kThreads) void decide_kernel(
    const float* logits, const float* q, const int32_t* drafts, const float* u, int k, int V, int nch,
    const float* cmax, const double* csum, int dstride, int doff, int32_t* out_tokens, int32_t* out_n,
    float* out_lp, FinalDraw* fin) {
  decide(logits, q, drafts, u, blockIdx.x, k, V, nch, cmax, csum, dstride, doff, true, out_tokens, out_n,
         out_lp, fin);
}

// ---- pass 3 ---------------------------------------------------------------------------
// Integer masses of chunk c of sequence b's final-draw row, per 256-logit sub-block. Logit t of
// the chunk sits at c*8192 + 2048 w + 256 i + 4 l + e for wavefront w, step i < 8, lane l, e < 4;
// sub-block 8 w + i is [256 (8 w + i), +256) of the chunk. A workgroup takes kMassSteps of the
// steps. The pass is bound by its ~30 instructions per logit and their latency, so it is cut small:
// with all 8 steps in one workgroup a wavefront alone took 9.5 us (one sequence, vocabulary 151936;
// with 2 steps 4.0), and 128 sequences ended 1 us later. kDecide: every workgroup takes its
// sequence's decisions for itself instead of reading them (the first of them stores them, all but the
// tokens: out_tokens may be the array that the others read the drafts from), which saves a launch where the chip is mostly empty anyway (one sequence: 4.8 + 4.0 us and the gap
// between the launches against 7.9); with 128 sequences it costs 7 us.
constexpr int kMassSteps = 2;
constexpr int kMassParts = 8 / kMassSteps;
template <bool kVec, bool kDecide>
__global__ __launch_bounds__(kThreads) void mass_kernel(
    const float* __restrict__ logits, const float* __restrict__ q, const int32_t* __restrict__ drafts,
    const float* __restrict__ u, int B, int k, int V, int nch, const float* __restrict__ cmax,
    const double* __restrict__ csum, int dstride, int doff, int32_t* __restrict__ out_n,
    float* __restrict__ out_lp, FinalDraw* __restrict__ fin, unsigned long long* __restrict__ sub_tot) {
  __shared__ double s_tab[256];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  for (long id = blockIdx.x; id < long(B) * nch * kMassParts; id += gridDim.x) {
    const int part = int(id % kMassParts);
    const int b = int(id / kMassParts / nch), c = int(id / kMassParts % nch);
    const long r0 = long(b) * (k + 1);
    FinalDraw f;
    if constexpr (kDecide)
      f = decide(logits, q, drafts, u, b, k, V, nch, cmax, csum, dstride, doff, c == 0 && part == 0,
                 nullptr, out_n, out_lp, fin);
    else f = fin[b];
    const float* lrow = logits + (r0 + f.row) * V;
    const float* qrow = f.mode == 1 ? q + (long(b) * k + f.row) * V : nullptr;
    const int t_base = c * kChunk + 2048 * wave + kSub * kMassSteps * part + 4 * lane;
    Quad qd[kMassSteps];
#pragma unroll
    for (int i = 0; i < kMassSteps; ++i) quad_load<kVec>(lrow, qrow, t_base + kSub * i, V, f.mode, qd[i]);
    __syncthreads();                                 // the last round is done with the table
    exp_table_init(s_tab, 1.0 / f.S, threadIdx.x, kThreads);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kMassSteps; ++i) {
      unsigned long long g[4];
      const unsigned long long sb = wave_sum_dpp(quad_mass(qd[i], t_base + kSub * i, V, f, f.mode, s_tab, g));
      if (lane == 0) sub_tot[(long(b) * nch + c) * kSubs + 8 * wave + kMassSteps * part + i] = sb;
    }
  }
}

// ---- pass 4 ---------------------------------------------------------------------------
// One wavefront per sequence. Zero residual mass (p <= q everywhere after rounding) falls
// back to p: the chunk and sub-block masses of p are then recomputed here (rare path). kDecide: the
// sequence's accepted drafts (k < 64) are stored here too, read and written by one instruction each, as
// out_tokens may overlap them.
template <bool kVec, bool kDecide>
__global__ __launch_bounds__(kWave) void draw_pick_kernel(
    const float* __restrict__ logits, const float* __restrict__ q, const int32_t* drafts,
    const float* __restrict__ u, int k, int V, int nch, int dstride, int doff,
    const FinalDraw* __restrict__ fin, const unsigned long long* __restrict__ sub_tot, int32_t* out_tokens,
    float* __restrict__ out_lp) {
  __shared__ double s_tab[256];
  const int b = blockIdx.x;
  const int lane = threadIdx.x;
  const FinalDraw f = fin[b];
  int draft = -1;
  if (kDecide && lane < f.row) draft = drafts[long(b) * dstride + doff + lane];
  exp_table_init(s_tab, 1.0 / f.S, lane, kWave);
  __syncthreads();
  const float* lrow = logits + (long(b) * (k + 1) + f.row) * V;
  const float* qrow = f.mode == 1 ? q + (long(b) * k + f.row) * V : nullptr;
  const unsigned long long* subs = sub_tot + long(b) * nch * kSubs;
  // mass of chunk c: its sub-blocks', two per load
  auto chunk_mass = [&](int c) {
    typedef unsigned long long Pair __attribute__((ext_vector_type(2)));
    Pair v = {0ull, 0ull};
#pragma unroll
    for (int j = 0; j < kSubs / 2; ++j) v += reinterpret_cast<const Pair*>(subs + long(c) * kSubs)[j];
    return v[0] + v[1];
  };
  const float ub = u[long(b) * (k + 1) + k];
  unsigned long long tot = 0;
  unsigned long long mine0 = 0;                       // of chunk `lane`
  for (int c = lane; c < nch; c += kWave) {
    const unsigned long long v = chunk_mass(c);
    if (c == lane) mine0 = v;
    tot += v;
  }
  tot = wave_sum(tot);
  int mode = f.mode;
  // sum of the masses of sub-block j of chunk c under `mode`, recomputed by the wavefront
  auto sub_mass = [&](int c, int j, int md) {
    unsigned long long g[4];
    const int t0 = c * kChunk + kSub * j + 4 * lane;
    Quad d;
    quad_load<kVec>(lrow, qrow, t0, V, md, d);
    return wave_sum(quad_mass(d, t0, V, f, md, s_tab, g));
  };
  if (tot == 0 && mode != 0) {
    mode = 0;
    tot = 0;
    for (int c = 0; c < nch; ++c)
      for (int j = 0; j < kSubs; ++j) tot += sub_mass(c, j, 0);
  }
  const unsigned long long u32 = (unsigned long long)(double(ub) * 4294967296.0);
  // target = (tot * u32) >> 32 without a 128-bit type
  const unsigned long long target = (tot >> 32) * u32 + (((tot & 0xffffffffull) * u32) >> 32);
  // 1. the chunk holding the target
  unsigned long long pre = 0;   // mass before the current window
  int chunk = -1;
  for (int c0 = 0; c0 < nch && chunk < 0; c0 += kWave) {
    const int c = c0 + lane;
    unsigned long long v = 0;
    if (mode == f.mode) {
      if (c < nch) v = c0 == 0 ? mine0 : chunk_mass(c);
    } else {
      // fallback: chunk masses of p, one chunk at a time (wavefront-wide sums)
      for (int cc = c0; cc < min(nch, c0 + kWave); ++cc) {
        unsigned long long sm = 0;
        for (int j = 0; j < kSubs; ++j) sm += sub_mass(cc, j, 0);
        if (lane == cc - c0) v = sm;
      }
    }
    const unsigned long long incl = wave_incl_scan(v, lane);
    const unsigned long long hit = __ballot(c < nch && pre + incl > target);
    if (hit) {
      const int l = __builtin_ctzll(hit);
      chunk = c0 + l;
      pre += __shfl(incl - v, l, kWave);
    } else {
      pre += __shfl(incl, kWave - 1, kWave);
    }
  }
  int token = -1;
  if (chunk >= 0) {
    // 2. the sub-block inside the chunk (lanes 0..31 hold the 32 sub-block masses)
    unsigned long long v = 0;
    if (mode == f.mode) {
      if (lane < kSubs) v = subs[long(chunk) * kSubs + lane];
    } else {
      for (int j = 0; j < kSubs; ++j) {
        const unsigned long long s = sub_mass(chunk, j, 0);
        if (lane == j) v = s;
      }
    }
    unsigned long long incl = wave_incl_scan(v, lane);
    unsigned long long hit = __ballot(lane < kSubs && pre + incl > target);
    if (hit) {
      const int j = __builtin_ctzll(hit);
      pre += __shfl(incl - v, j, kWave);
      // 3. four logits per lane inside the sub-block
      unsigned long long g[4];
      const int t0 = chunk * kChunk + kSub * j + 4 * lane;
      Quad d;
      quad_load<kVec>(lrow, qrow, t0, V, mode, d);
      const unsigned long long mine = quad_mass(d, t0, V, f, mode, s_tab, g);
      incl = wave_incl_scan(mine, lane);
      hit = __ballot(pre + incl > target);
      if (hit) {
        const int l = __builtin_ctzll(hit);
        if (lane == l) {
          unsigned long long run = pre + incl - mine;
          for (int e = 0; e < 4; ++e) {
            run += g[e];
            if (run > target) {
              token = t0 + e;
              break;
            }
          }
        }
        token = __shfl(token, l, kWave);
      }
    }
  }
  if (kDecide) {
    if (lane <= k) out_tokens[long(b) * (k + 1) + lane] = lane == f.row ? token : draft;
  } else if (lane == 0) {
    out_tokens[long(b) * (k + 1) + f.row] = token;
  }
  if (lane == 0 && out_lp)
    out_lp[long(b) * (k + 1) + f.row] =
        token >= 0 ? float((double(lrow[token]) - f.m) - log(f.S)) : __builtin_nanf("");
}


// ---- MTP draft draws --------------------------------------------------------------------
// q[b * q_stride + t] = softmax(logits[b])_t in f32: (m, S) combined from the chunk
// statistics exactly as the accept decisions combine them, exp(l - m) by the table exp.
template <bool kVec>
__global__ __launch_bounds__(kThreads) void softmax_write_kernel(const float* __restrict__ logits,
                                                                 int V, int nch,
                                                                 const float* __restrict__ cmax,
                                                                 const double* __restrict__ csum,
                                                                 float* __restrict__ q, long q_stride) {
  __shared__ double tab[256];
  __shared__ double s_m, s_inv;
  const long row = blockIdx.x / nch;
  const int c = int(blockIdx.x % nch);
  if (threadIdx.x < kWave) {
    const int lane = threadIdx.x;
    float mx = -INFINITY;
    for (int cc = lane; cc < nch; cc += kWave) mx = fmaxf(mx, cmax[row * nch + cc]);
    mx = wave_max(mx);
    double acc = 0.0;
    for (int cc = lane; cc < nch; cc += kWave) {
      const float v = cmax[row * nch + cc];
      if (v != -INFINITY) acc += csum[row * nch + cc] * exp(double(v) - double(mx));
    }
    acc = wave_sum(acc);
    if (lane == 0) {
      s_m = double(mx);
      s_inv = 1.0 / acc;
    }
  }
  __syncthreads();
  const double m = s_m, inv = s_inv;
  exp_table_init(tab, 1.0, threadIdx.x, kThreads);
  __syncthreads();
  // 1 / S as a factor and not in the table: a sum that is not a number stays one in q
  auto prob = [&](float l) { return float(exp_nonpos(fmax(double(l) - m, kExpMin), tab) * inv); };
  const float* src = logits + row * long(V) + long(c) * kChunk;
  float* dst = q + row * q_stride + long(c) * kChunk;
  const int n = min(kChunk, V - c * kChunk);
  if (kVec) {
#pragma unroll 2
    for (int i = 0; i < kPerThread / 4; ++i) {
      const int e0 = 4 * (threadIdx.x + kThreads * i);
      if (e0 >= n) break;
      const floatx4_t l = __builtin_nontemporal_load(reinterpret_cast<const floatx4_t*>(src + e0));
      floatx4_t o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = prob(l[e]);
      *reinterpret_cast<floatx4_t*>(dst + e0) = o;
    }
  } else {
    for (int e = threadIdx.x; e < n; e += kThreads)
      dst[e] = prob(src[e]);
  }
}

// out[b] = the first index of the largest logit of row b (0 for a row with no finite max)
__global__ __launch_bounds__(kThreads) void argmax_kernel(const float* __restrict__ logits, int V,
                                                          int32_t* __restrict__ out) {
  __shared__ float s_v[kThreads / kWave];
  __shared__ int s_i[kThreads / kWave];
  const long row = blockIdx.x;
  const float* src = logits + row * long(V);
  float best = -INFINITY;
  int bi = V;
  for (int t = threadIdx.x; t < V; t += kThreads) {   // a thread's indices increase
    const float v = src[t];
    if (v > best) { best = v; bi = t; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(best, o, kWave);
    const int oi = __shfl_xor(bi, o, kWave);
    if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
  }
  const int w = threadIdx.x / kWave;
  if (threadIdx.x % kWave == 0) { s_v[w] = best; s_i[w] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int j = 1; j < kThreads / kWave; ++j)
      if (s_v[j] > best || (s_v[j] == best && s_i[j] < bi)) { best = s_v[j]; bi = s_i[j]; }
    out[row] = bi < V ? bi : 0;
  }
}


// ---- scores of given tokens -------------------------------------------------------------
// lp[r] = (l[r, y] - m) - ln S for y = targets[r] in [0, V), else NaN: one wavefront per row,
// (m, S) combined from the chunk statistics exactly as the accept decisions combine them,
// so that a recompute of emitted tokens reproduces the recorded log-probs bit for bit.
__global__ __launch_bounds__(kWave) void token_logprob_kernel(const float* __restrict__ logits,
                                                              int V, int nch,
                                                              const float* __restrict__ cmax,
                                                              const double* __restrict__ csum,
                                                              const int32_t* __restrict__ targets,
                                                              float* __restrict__ out) {
  const long row = blockIdx.x;
  const int lane = threadIdx.x;
  float mx = -INFINITY;
  for (int cc = lane; cc < nch; cc += kWave) mx = fmaxf(mx, cmax[row * nch + cc]);
  mx = wave_max(mx);
  double acc = 0.0;
  for (int cc = lane; cc < nch; cc += kWave) {
    const float v = cmax[row * nch + cc];
    if (v != -INFINITY) acc += csum[row * nch + cc] * exp(double(v) - double(mx));
  }
  acc = wave_sum(acc);
  if (lane == 0) {
    const int y = targets[row];
    out[row] = (y >= 0 && y < V)
                   ? float((double(logits[row * long(V) + y]) - double(mx)) - log(acc))
                   : __builtin_nanf("");
  }
}

}  // namespace

int sampler_chunk_elems() { return kChunk; }

size_t sampler_ws_bytes(int B, int k, int V) {
  const long nch = (V + kChunk - 1) / kChunk;
  const long rows = long(B) * (k + 1);
  Carver c(nullptr, 0);
  c.take<float>(rows * nch);
  c.take<double>(rows * nch);
  c.take<FinalDraw>(B);
  c.take<unsigned long long>(long(B) * nch);          // unused; part of the documented need
  c.take<unsigned long long>(long(B) * nch * kSubs);
  return c.used + 256;
}

hipError_t launch_spec_accept(const float* logits, const float* q, const int32_t* drafts,
                              const float* u, int B, int k, int V, int32_t* out_tokens,
                              int32_t* out_n, float* out_lp, void* ws, hipStream_t s,
                              int draft_stride, int draft_offset) {
  const int nch = (V + kChunk - 1) / kChunk;
  const long rows = long(B) * (k + 1);
  Carver c(ws, 0);
  float* cmax = c.take<float>(rows * nch);
  double* csum = c.take<double>(rows * nch);
  FinalDraw* fin = c.take<FinalDraw>(B);
  unsigned long long* stot = c.take<unsigned long long>(long(B) * nch * kSubs);
  const bool vec = (V % 4 == 0) && ((reinterpret_cast<uintptr_t>(logits) & 15) == 0) &&
                   (q == nullptr || (reinterpret_cast<uintptr_t>(q) & 15) == 0);
  const int ds = draft_stride < 0 ? k : draft_stride;
  const dim3 g1{unsigned(rows * nch)}, g3{unsigned(B)};
  // (2^22 workgroups at most, each taking several parts past that)
  const long parts = long(B) * nch * kMassParts;
  const dim3 g2{unsigned(parts < (1L << 22) ? parts : 1L << 22)};
  const bool few = parts <= 512 && k < kRowsPerBatch;   // two workgroups a CU, one batch of rows
  auto run = [&](auto vec_c) {
    constexpr bool kVec = decltype(vec_c)::value;
    chunk_stats_kernel<kVec><<<g1, kThreads, 0, s>>>(logits, rows, V, nch, cmax, csum);
    if (few) {
      mass_kernel<kVec, true><<<g2, kThreads, 0, s>>>(logits, q, drafts, u, B, k, V, nch, cmax, csum, ds,
                                                      draft_offset, out_n, out_lp, fin, stot);
      draw_pick_kernel<kVec, true><<<g3, kWave, 0, s>>>(logits, q, drafts, u, k, V, nch, ds, draft_offset, fin,
                                                        stot, out_tokens, out_lp);
    } else {
      decide_kernel<<<g3, kThreads, 0, s>>>(logits, q, drafts, u, k, V, nch, cmax, csum, ds,
                                            draft_offset, out_tokens, out_n, out_lp, fin);
      mass_kernel<kVec, false><<<g2, kThreads, 0, s>>>(logits, q, drafts, u, B, k, V, nch, cmax, csum, ds,
                                                       draft_offset, out_n, out_lp, fin, stot);
      draw_pick_kernel<kVec, false><<<g3, kWave, 0, s>>>(logits, q, drafts, u, k, V, nch, ds, draft_offset, fin,
                                                         stot, out_tokens, out_lp);
    }
  };
  if (vec) run(std::true_type{});
  else run(std::false_type{});
  return hipGetLastError();
}

size_t draft_draw_ws_bytes(int B, int V) {
  Carver c(nullptr, 0);
  c.take<uint8_t>(sampler_ws_bytes(B, 0, V));
  c.take<int32_t>(B);
  c.take<float>(B);
  return c.used + 256;
}

hipError_t launch_draft_draw(const float* logits, int B, int V, const float* u, int32_t* out_tok,
                             float* q_out, long q_stride, void* ws, hipStream_t s) {
  if (u == nullptr) {
    argmax_kernel<<<B, kThreads, 0, s>>>(logits, V, out_tok);
    return hipGetLastError();
  }
  Carver c(ws, 0);
  void* samp = c.take<uint8_t>(sampler_ws_bytes(B, 0, V));
  int32_t* n = c.take<int32_t>(B);
  float* lp = c.take<float>(B);
  // a draw from p is the bonus draw of a step without drafts (k = 0, one uniform per row)
  hipError_t e = launch_spec_accept(logits, nullptr, out_tok, u, B, 0, V, out_tok, n, lp, samp, s);
  if (e != hipSuccess || q_out == nullptr) return e;
  // the row statistics of pass 1 sit at the start of the sampler's workspace
  const int nch = (V + kChunk - 1) / kChunk;
  Carver cs(samp, 0);
  const float* cmax = cs.take<float>(long(B) * nch);
  const double* csum = cs.take<double>(long(B) * nch);
  const bool vec = (V % 4 == 0) && (q_stride % 4 == 0) &&
                   ((reinterpret_cast<uintptr_t>(logits) & 15) == 0) &&
                   ((reinterpret_cast<uintptr_t>(q_out) & 15) == 0);
  const dim3 g{unsigned(long(B) * nch)};
  if (vec) softmax_write_kernel<true><<<g, kThreads, 0, s>>>(logits, V, nch, cmax, csum, q_out, q_stride);
  else softmax_write_kernel<false><<<g, kThreads, 0, s>>>(logits, V, nch, cmax, csum, q_out, q_stride);
  return hipGetLastError();
}

size_t token_logprob_ws_bytes(long rows, int V) {
  const long nch = (V + kChunk - 1) / kChunk;
  Carver c(nullptr, 0);
  c.take<float>(rows * nch);
  c.take<double>(rows * nch);
  return c.used + 256;
}

hipError_t launch_token_logprobs(const float* logits, long rows, int V, const int32_t* targets,
                                 float* out, void* ws, hipStream_t s) {
  const int nch = (V + kChunk - 1) / kChunk;
  Carver c(ws, 0);
  float* cmax = c.take<float>(rows * nch);
  double* csum = c.take<double>(rows * nch);
  const bool vec = (V % 4 == 0) && ((reinterpret_cast<uintptr_t>(logits) & 15) == 0);
  const dim3 g1{unsigned(rows * nch)}, g2{unsigned(rows)};
  if (vec) chunk_stats_kernel<true><<<g1, kThreads, 0, s>>>(logits, rows, V, nch, cmax, csum);
  else chunk_stats_kernel<false><<<g1, kThreads, 0, s>>>(logits, rows, V, nch, cmax, csum);
  token_logprob_kernel<<<g2, kWave, 0, s>>>(logits, V, nch, cmax, csum, targets, out);
  return hipGetLastError();
}

}  // namespace molt
