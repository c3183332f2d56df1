// post.hip -- the polar-image epilogue on CDNA4 (gfx950): range blur
// (measurement noise), uniform system noise, gradient-noise ambient noise,
// dB and 8-bit map (Sec. III-B "Polar Image", Sec. III-C "Noise").
//
// One workgroup takes 1024 range bins of one azimuth column; each lane
// produces four consecutive pixels.  The workgroup issues all its global
// loads first, builds the table of lattice gradients its bins need while they
// are in flight, then stages the column segment plus the blur halo in LDS as
// float64.  Everything is float64 in a fixed order.
//
// What bounds it: vector issue (a float64 or 64-bit multiply-add instruction
// takes 4.5 clocks of a SIMD, so a pixel's instructions take longer than its
// nine bytes of HBM traffic), hence fused multiply-adds, the blur's taps read
// two at a time, divisions by the lattice spacing as multiplications with a
// correction, a logarithm by table, and nothing in scratch memory.  64 images
// of 400 x 3776 with every term on: 0.700 -> 0.436 ms (1.24 -> 2.00 TB/s); HBM
// alone would take 0.18.  The gradient table takes 16 bytes a lattice point:
// with a lattice of one bin and a blur a block holds 44 KB of LDS, three blocks
// per CU, and is still ahead of the plain form it replaced (1.69 -> 1.64 ms at
// sigma 2; 0.96 -> 0.68 with a lattice of four bins).
#include <hip/hip_runtime.h>

#include "philox.h"
#include "post.h"
#include "rr_internal.h"

#pragma clang fp contract(off)

namespace rr {

namespace {

// e + amp * (x >> 11) 2^-53: the 53 bits as their upper 32 and lower 21,
// whose sum is exact
__device__ __forceinline__ double add_uniform(double e, double amp, uint64_t x) {
  const double hi = (double)(uint32_t)(x >> 32), lo = (double)((uint32_t)x >> 11);
  return __builtin_fma(amp, __builtin_fma(hi, 1.0 / 4294967296.0, lo * (1.0 / 9007199254740992.0)), e);
}

// quintic fade of improved gradient noise (Perlin, SIGGRAPH 2002)
__device__ __forceinline__ double fade5(double t) {
  return t * t * t * __builtin_fma(t, __builtin_fma(t, 6.0, -15.0), 10.0);
}

// a / b for an integer a <= 65535, given r = 1 / b correctly rounded: the
// product is within one ulp and the correction makes it the correctly
// rounded quotient (Markstein, "Computation of elementary functions on the
// IBM RISC System/6000 processor", 1990)
__device__ __forceinline__ double div_by(double a, double b, double r) {
  const double q = a * r;
  return __builtin_fma(__builtin_fma(-q, b, a), r, q);
}

// a b + c with the constant c in a scalar register pair (as an accumulator it
// would be copied to vector registers first, two more instructions)
__device__ __forceinline__ double fma_c(double a, double b, double c) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
  return r;
}

// 10 log10 by table.  e = 2^k z with z in [11/16, 11/8); interval i of the
// leading bits of z has an approximate reciprocal v (1 around z = 1, so that
// the result keeps its relative accuracy there) and -10 log10(v); with
// u = z v - 1, |u| <= 2^-7, the rest is the series of log1p to u^8 (relative
// truncation error below 2^-58).  Largest relative error 2.2e-16 on 20,000
// values over 1e-60..1e10 and around 1.
struct LogEntry {
  double v, l;
};
__device__ const LogEntry kLogTable[128] = {
    {1.4504249291784703, -1.6149525558800821}, {1.4422535211267606, -1.590416079207367},
    {1.4341736694677871, -1.5660174486363756}, {1.426183844011142, -1.5417551239751162},
    {1.4182825484764543, -1.5176275907017283}, {1.4104683195592287, -1.4936333593971824},
    {1.4027397260273973, -1.4697709651935607}, {1.3950953678474114, -1.446038967237414},
    {1.3875338753387534, -1.4224359481677038}, {1.3800539083557952, -1.3989605136078491},
    {1.3726541554959786, -1.3756112916714316}, {1.3653333333333333, -1.3523869324811189},
    {1.3580901856763925, -1.3292861077003788}, {1.3509234828496042, -1.306307510077584},
    {1.3438320209973753, -1.2834498530021146}, {1.3368146214099217, -1.2607118700720803},
    {1.3298701298701299, -1.2380923146733007}, {1.322997416020672, -1.2155899595691937},
    {1.3161953727506426, -1.19320359650123}, {1.3094629156010231, -1.1709320357996398},
    {1.3027989821882953, -1.1487741060040408}, {1.2962025316455696, -1.1267286534937053},
    {1.2896725440806045, -1.1047945421271568}, {1.2832080200501252, -1.082970652890825},
    {1.2768079800498753, -1.0612558835564845}, {1.2704714640198511, -1.039649148347213},
    {1.2641975308641975, -1.018149377611622}, {1.257985257985258, -0.9967555175061071},
    {1.2518337408312958, -0.9754665296848896}, {1.245742092457421, -0.9542813909976157},
    {1.2397094430992737, -0.9331990931942976}, {1.2337349397590363, -0.9122186426373808},
    {1.2278177458033572, -0.891339060020732}, {1.2219570405727924, -0.8705593800953547},
    {1.2161520190023754, -0.8498786514016247}, {1.210401891252955, -0.8292959360078841},
    {1.204705882352941, -0.8088103092551918}, {1.199063231850117, -0.788420859508069},
    {1.1934731934731935, -0.7681266879110651}, {1.1879350348027842, -0.7479269081509914},
    {1.1824480369515011, -0.727820646224653}, {1.1770114942528735, -0.7078070402119342},
    {1.17162471395881, -0.6878852400540891}, {1.1662870159453302, -0.6680544073370936},
    {1.1609977324263039, -0.6483137150799223}, {1.1557562076749435, -0.6286623475276116},
    {1.150561797752809, -0.609099499948992}, {1.145413870246085, -0.5896243784389427},
    {1.1403118040089086, -0.5702361997250757}, {1.1352549889135255, -0.5509341909787022},
    {1.130242825607064, -0.5317175896299888}, {1.1252747252747253, -0.5125856431871835},
    {1.1203501094091903, -0.4935376090598052}, {1.1154684095860568, -0.47457275438569557},
    {1.1106290672451193, -0.45569035586182627}, {1.1058315334773219, -0.4368896995787765},
    {1.1010752688172043, -0.41817008085876833}, {1.0963597430406853, -0.39953080409718617},
    {1.091684434968017, -0.3809711826074748}, {1.0870488322717622, -0.36249053846934576},
    {1.0824524312896406, -0.34408820238019205}, {1.0778947368421052, -0.3257635135096418},
    {1.0733752620545074, -0.3075158193571686}, {1.068893528183716, -0.28934447561267496},
    {1.0644490644490645, -0.27124884601999016}, {1.060041407867495, -0.25322830224318643},
    {1.0556701030927835, -0.2352822237356711}, {1.051334702258727, -0.21740999761196442},
    {1.047034764826176, -0.19961101852210553}, {1.0427698574338085, -0.18188468852862244},
    {1.0385395537525355, -0.16423041698600735}, {1.0343434343434343, -0.14664762042262036},
    {1.0301810865191148, -0.12913572242498678}, {1.0260521042084167, -0.11169415352440806},
    {1.0219560878243512, -0.09432235108585003}, {1.0178926441351888, -0.07701975919903316},
    {1.0138613861386139, -0.05978582857169383}, {1.009861932938856, -0.04262001642494803},
    {1.005893909626719, -0.025521786390719794}, {1.0, 0.0},
    {1.0, 0.0}, {0.9884169884169884, 0.05059798769402256},
    {0.9808429118773946, 0.08400542026431422}, {0.973384030418251, 0.1171578317790831},
    {0.9660377358490566, 0.15005908624958286}, {0.9588014981273408, 0.18271296052725655},
    {0.9516728624535316, 0.2151231469055844}, {0.9446494464944649, 0.24729325562556181},
    {0.9377289377289377, 0.27922681728906473}, {0.9309090909090909, 0.3109272851841309},
    {0.924187725631769, 0.34239803752598974}, {0.9175627240143369, 0.3736423796174799},
    {0.9110320284697508, 0.4046635459323035}, {0.9045936395759717, 0.4354647021244068},
    {0.8982456140350877, 0.4660489469666063}, {0.89198606271777, 0.49641931422142765},
    {0.8858131487889274, 0.5265787744469829}, {0.8797250859106529, 0.5565302367405773},
    {0.8737201365187713, 0.5862765504225989}, {0.8677966101694915, 0.6158205066631345},
    {0.8619528619528619, 0.6451648400536281}, {0.8561872909698997, 0.674312230125801},
    {0.8504983388704319, 0.7032653028199378}, {0.8448844884488449, 0.7320266319045544},
    {0.839344262295082, 0.7605987403493628}, {0.8338762214983714, 0.7889841016533691},
    {0.8284789644012945, 0.8171851411298506}, {0.8231511254019293, 0.8452042371498795},
    {0.8178913738019169, 0.8730437223459894}, {0.8126984126984127, 0.9007058847775095},
    {0.807570977917981, 0.9281929690590195}, {0.8025078369905956, 0.9555071774533158},
    {0.7975077881619937, 0.9826506709302253}, {0.7925696594427245, 1.009625570192533},
    {0.7876923076923077, 1.036433956670248}, {0.7828746177370031, 1.063077873484365},
    {0.7781155015197568, 1.0895593263812473}, {0.7734138972809668, 1.1158802846386917},
    {0.7687687687687688, 1.1420426819447032}, {0.764179104477612, 1.1680484172499568},
    {0.7596439169139466, 1.1938993555948905}, {0.7551622418879056, 1.219597328912326},
    {0.750733137829912, 1.2451441368064815}, {0.7463556851311953, 1.2705415473092094},
    {0.7420289855072464, 1.2957912976142456}, {0.7377521613832853, 1.3208950947902418},
    {0.7335243553008596, 1.3458546164733034}, {0.7293447293447294, 1.370671511539745},
};
// finite normal e > 0
__device__ __forceinline__ double ten_log10(double e, const LogEntry* table) {
  const uint32_t hi = (uint32_t)__double2hiint(e);
  const uint32_t t = hi - 0x3fe60000u;
  const LogEntry en = table[(t >> 13) & 127u];
  const double k = (double)((int32_t)t >> 20);
  const double z = __hiloint2double((int)(hi - (t & 0xfff00000u)), __double2loint(e));
  const double u = __builtin_fma(z, en.v, -1.0);
  // 10 / ln(10) (-1)^(n + 1) / n
  double p = __builtin_fma(u, -0.5428681023790648, 0.6204206884332168);
  p = fma_c(p, u, -0.7238241365054197);
  p = fma_c(p, u, 0.8685889638065036);
  p = fma_c(p, u, -1.0857362047581296);
  p = fma_c(p, u, 1.4476482730108393);
  p = fma_c(p, u, -2.171472409516259);
  p = fma_c(p, u, 4.342944819032518);
  return __builtin_fma(k, 3.010299956639812, __builtin_fma(p, u, en.l));
}

// lattice gradient g in 0..7: (1,1), (-1,1), (1,-1), (-1,-1), (1,0), (-1,0),
// (0,1), (0,-1)
__device__ __forceinline__ float2 lattice_gradient(uint32_t g) {
  float gx = g < 6u ? ((g & 1u) ? -1.0f : 1.0f) : 0.0f;
  float gy = g < 4u ? ((g & 2u) ? -1.0f : 1.0f) : (g < 6u ? 0.0f : ((g & 1u) ? -1.0f : 1.0f));
  return make_float2(gx, gy);
}

// gradient table entry of a lattice point: its x component times the
// distance from the lattice column to this azimuth (exact), and its y
// component
struct GradEntry {
  double ax, gy;
};

// energy of cell j of the image (or of the fixed-point accumulator, as the
// scan's finalize converts it)
template <bool kFromAcc>
__device__ __forceinline__ float load_cell(const PostArgs& a, size_t j) {
  if constexpr (kFromAcc)
    return (float)((double)a.acc[j] * kFixedInv);
  else
    return a.img[j];
}

template <bool kFromAcc>
__global__ __launch_bounds__(kPostBlock) void k_post(PostArgs a) {
  extern __shared__ double smem[];
  LogEntry* logs = reinterpret_cast<LogEntry*>(smem);             // [128]
  GradEntry* grad = reinterpret_cast<GradEntry*>(smem + 2 * 128);  // [2][gcap]
  double* tile = smem + 2 * 128 + 4u * a.gcap;                      // [kPostTile + 2R], 16-byte aligned
  const uint32_t b0 = blockIdx.x * (uint32_t)kPostTile;
  const uint32_t k = blockIdx.y, img = blockIdx.z;
  const uint32_t nb = min((uint32_t)kPostTile, a.n_bins - b0);
  const int R = a.R;
  const size_t row = ((size_t)img * a.n_az + k) * a.n_bins;
  const uint32_t tid = threadIdx.x;
  // lane t takes the four consecutive bins 4t..4t+3 of the tile: they share
  // one generator block (word s for bin 4t + s) and one 16-byte store
  const uint32_t q0 = 4u * tid;
  const uint32_t nq = q0 < nb ? min(4u, nb - q0) : 0u;
  const uint32_t bq = b0 + q0;
  const size_t o = row + bq;

  // 1. every global load of the block is issued before anything waits on it:
  //    the lane's own four cells and, for lanes below 2R, one halo cell
  // (branch-free: lanes past the tile's end re-read an in-bounds cell and
  // drop it, so the compiler places no wait before the gradient table)
  float c[4];
  if (!kFromAcc && (a.n_bins & 3u) == 0u && (reinterpret_cast<uintptr_t>(a.img) & 15u) == 0u) {
    // rows of whole, aligned groups of four: one load (a group is full or empty)
    const float4 v = *reinterpret_cast<const float4*>(a.img + (nq ? o : row + b0));
    c[0] = v.x;
    c[1] = v.y;
    c[2] = v.z;
    c[3] = v.w;
  } else {
    const uint32_t last = nq ? nq - 1u : 0u;
    const size_t base = nq ? o : row + b0;
    // (c[t] for t >= nq is a duplicate that no store uses)
#pragma unroll
    for (uint32_t t = 0; t < 4u; ++t) c[t] = load_cell<kFromAcc>(a, base + min(t, last));
  }
  const bool has_halo = (int)tid < 2 * R;
  const long hb = (int)tid < R ? (long)b0 - R + (long)tid : (long)b0 + (long)nb + (long)tid - R;
  const bool halo_in = has_halo && hb >= 0 && hb < (long)a.n_bins;
  const size_t hcell = row + (size_t)(halo_in ? hb : (long)b0);
  const float hv = load_cell<kFromAcc>(a, hcell);
  const float h = halo_in ? hv : 0.0f;
  const int hslot = has_halo ? ((int)tid < R ? (int)tid : R + (int)nb + (int)tid - R) : -1;

  // (as one struct the entry would go through scratch memory: 454 -> 431 us
  // for the 64 images)
  double log_v = 0.0, log_l = 0.0;
  if (tid < 128u) {
    log_v = kLogTable[tid].v;
    log_l = kLogTable[tid].l;
  }

  // 2. gradient noise: lattice columns i0, i0 + 1 and rows jlo..jhi of this
  //    tile, computed while the loads are in flight
  const bool perlin = a.pamp > 0.0;
  // (lattice coordinates fit in int: k, b <= 65535 and the cells are >= 1)
  const double x = div_by((double)k, a.cell_az, a.rcell_az);
  const double fx0 = floor(x);
  const double fx = x - fx0;
  const int i0 = (int)fx0;
  const int jlo = (int)floor(div_by((double)b0, a.cell_bins, a.rcell_bins));
  const uint32_t scan = a.scan_id + img;
  if (perlin) {
    const int jhi = (int)floor(div_by((double)(b0 + nb - 1u), a.cell_bins, a.rcell_bins)) + 1;
    // the host sizes gcap for the longest row range a tile can span
    const uint32_t cnt = min((uint32_t)(jhi - jlo + 1), a.gcap);
    for (uint32_t t = tid; t < 2u * cnt; t += kPostBlock) {
      uint32_t side = t / cnt, jj = t - side * cnt;
      uint64_t r[4];
      philox4x64_10(a.seed, (uint64_t)scan, (uint64_t)(int64_t)(i0 + (int)side),
                    (uint64_t)(int64_t)(jlo + (int)jj), 2u, 0u, r);
      const float2 v = lattice_gradient((uint32_t)(r[0] >> 61));
      grad[side * a.gcap + jj] = GradEntry{(double)v.x * (side ? fx - 1.0 : fx), (double)v.y};
    }
  }

  if (tid < 128u) logs[tid] = LogEntry{log_v, log_l};

  // 3. the scan's float image, and the blur's LDS tile with its halo
  if constexpr (kFromAcc) {
    if (a.image) {
      if (nq == 4u && (reinterpret_cast<uintptr_t>(a.image + o) & 15u) == 0u) {
        *reinterpret_cast<float4*>(a.image + o) = make_float4(c[0], c[1], c[2], c[3]);
      } else {
        for (uint32_t t = 0; t < nq; ++t) a.image[o + t] = c[t];
      }
    }
  }
  if (R > 0) {
#pragma unroll
    for (uint32_t t = 0; t < 4u; ++t)
      if (t < nq) tile[(uint32_t)R + q0 + t] = (double)c[t];
    if (hslot >= 0) tile[hslot] = (double)h;
  }
  __syncthreads();
  if (nq == 0u) return;

  // 4. measurement noise: taps m = 0..2R of tile[q0 + t + m] for bin q0 + t,
  //    each pixel summing its taps in order; a sliding window reads each tile
  //    entry once, two per LDS access
  double e[4];
  if (R == 0) {
#pragma unroll
    for (int t = 0; t < 4; ++t) e[t] = (double)c[t];
  } else {
    e[0] = e[1] = e[2] = e[3] = 0.0;
    const double2* tp = reinterpret_cast<const double2*>(tile + q0);
    double2 p0 = tp[0], p1 = tp[1];
#pragma unroll 3
    for (int m = 0; m < R; ++m) {
      const double2 p2 = tp[m + 2];
      const double wa = a.w[2 * m], wb = a.w[2 * m + 1];
      e[0] = __builtin_fma(wa, p0.x, e[0]);
      e[1] = __builtin_fma(wa, p0.y, e[1]);
      e[2] = __builtin_fma(wa, p1.x, e[2]);
      e[3] = __builtin_fma(wa, p1.y, e[3]);
      e[0] = __builtin_fma(wb, p0.y, e[0]);
      e[1] = __builtin_fma(wb, p1.x, e[1]);
      e[2] = __builtin_fma(wb, p1.y, e[2]);
      e[3] = __builtin_fma(wb, p2.x, e[3]);
      p0 = p1;
      p1 = p2;
    }
    const double wl = a.w[2 * R];
    e[0] = __builtin_fma(wl, p0.x, e[0]);
    e[1] = __builtin_fma(wl, p0.y, e[1]);
    e[2] = __builtin_fma(wl, p1.x, e[2]);
    e[3] = __builtin_fma(wl, p1.y, e[3]);
  }
  // 5. system noise
  if (a.uamp > 0.0) {
    uint64_t r[4];
    philox4x64_10<true>(a.seed, (uint64_t)scan, (uint64_t)k, (uint64_t)(bq >> 2), 1u, 0u, r);
#pragma unroll
    for (int t = 0; t < 4; ++t) e[t] = add_uniform(e[t], a.uamp, r[t]);
  }
  // 6. ambient noise
  if (perlin) {
    const double fu = fade5(fx);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const double y = div_by((double)(bq + (uint32_t)t), a.cell_bins, a.rcell_bins);
      const double fy0 = floor(y);
      // rows of the last (ragged) group beyond the tile stay inside the table
      const uint32_t jj = min((uint32_t)((int)fy0 - jlo), a.gcap - 2u);
      const double fy = y - fy0, fy1 = fy - 1.0;
      const GradEntry* g0 = grad + jj;
      const GradEntry* g1 = grad + a.gcap + jj;
      const double n00 = __builtin_fma(g0[0].gy, fy, g0[0].ax), n10 = __builtin_fma(g1[0].gy, fy, g1[0].ax);
      const double n01 = __builtin_fma(g0[1].gy, fy1, g0[1].ax), n11 = __builtin_fma(g1[1].gy, fy1, g1[1].ax);
      const double nx0 = __builtin_fma(fu, n10 - n00, n00);
      const double nx1 = __builtin_fma(fu, n11 - n01, n01);
      const double n = __builtin_fma(fade5(fy), nx1 - nx0, nx0);
      e[t] = __builtin_fma(a.pamp, __builtin_fma(0.5, n, 0.5), e[t]);
    }
  }
  // 7. dB and 8-bit pixel
  float db[4];
  uint32_t px[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    // normal and finite (a zero, negative, NaN, infinite or denormal energy
    // takes the branch)
    double L = ten_log10(e[t], logs);
    if ((uint32_t)__double2hiint(e[t]) - 0x00100000u >= 0x7fe00000u)
      L = e[t] > 0.0 ? 10.0 * log10(e[t]) : -__builtin_huge_val();
    // one multiply by max / (0 - floor) instead of the division: the
    // pixel value moves by a few ulp at most, far inside the 1e-9 band
    // around rounding boundaries where the two orders may disagree.  The
    // conversion truncates.
    px[t] = (uint32_t)fmin(fmax(__builtin_fma(L - a.db_floor, a.px_scale, 0.5), 0.0), a.max_value);
    db[t] = (float)L;
  }
  if (a.db) {
    float* d = a.db + o;
    if (nq == 4u && (reinterpret_cast<uintptr_t>(d) & 15u) == 0u)
      *reinterpret_cast<float4*>(d) = make_float4(db[0], db[1], db[2], db[3]);
    else
      for (uint32_t t = 0; t < nq; ++t) d[t] = db[t];
  }
  if (a.u8) {
    uint8_t* u = a.u8 + o;
    if (nq == 4u && (reinterpret_cast<uintptr_t>(u) & 3u) == 0u)
      *reinterpret_cast<uint32_t*>(u) =
          px[0] | (px[1] << 8) | (px[2] << 16) | (px[3] << 24);
    else
      for (uint32_t t = 0; t < nq; ++t) u[t] = (uint8_t)px[t];
  }
}

}  // namespace

hipError_t launch_post(const PostArgs& a, hipStream_t st) {
  if (a.n_az == 0 || a.n_bins == 0 || a.n_images == 0) return hipSuccess;
  dim3 grid((a.n_bins + kPostTile - 1) / kPostTile, a.n_az, a.n_images);
  const size_t lds = post_lds_bytes(a);
  if (a.acc)
    hipLaunchKernelGGL(k_post<true>, grid, dim3(kPostBlock), lds, st, a);
  else
    hipLaunchKernelGGL(k_post<false>, grid, dim3(kPostBlock), lds, st, a);
  return hipGetLastError();
}

}  // namespace rr
