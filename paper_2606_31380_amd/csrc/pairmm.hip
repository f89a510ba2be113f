// Inter-body pair sum with several right-hand sides on the matrix cores: the
// kernel matrix K_ij of a tile of targets and a chunk of sources is evaluated
// in registers (the per-pair arithmetic of pairsum.hip) and multiplied with
// the densities at once,
//   w_i[r] = sum_j K_ij mu_j[r],  K_ij = (1/4 pi)(ik r - 1) e^{ikr} / r^3
//                                        (aw_j . (y_j - x_i))   (double layer),
// so each pair's distance and phase serve every right-hand side and the
// complex products run on MFMA.  Needs k > 0 in every problem.
//
// Chunks of MM_C = 32 consecutive sources and tiles of 16 consecutive targets
// never straddle bodies or problems (a body has 16 n_panels n_theta nodes and
// n_theta is even), so the exclusion of pairs on one body is uniform over a
// wavefront and a chunk.
#include <algorithm>
#include <vector>

#include "fastmath.h"
#include "internal.h"

namespace qax {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- FP32 path
// Every FP32 factor x enters the FP16 matrix products as h + l, h = x rounded
// to FP16 and l = x - h rounded to FP16 (22 to 23 significant bits while x is
// above 2^-3 in size), and x y = h h' + h l' + l h' in FP32 (the dropped l l'
// is below 2^-22 of the product, of random sign).  Powers of two keep the
// factors in range: K is scaled per source body by S_b so that the largest
// entry that a target at least rho_b = R_b / 2 off the body's bounding ball
// (radius R_b) can have is below 2^14, for a tile of targets so far off that none
// can pass 2^4 by what brings that bound up to 2^14 as well, mu per source body and
// right-hand side by sigma so that its largest entry there is below 2^15.  Sums are taken out of
// these scales where the sources' body changes, so that a body's densities keep
// their digits beside another's larger ones, or ones that are not finite.
__device__ __forceinline__ void split2(float x0, float x1, uint32_t& h, uint32_t& l) {
  f32x2 r = {x0, x1};
  h = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, f16x2));
  // x - h from the packed halves, one mixed-precision fma each
  asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r[0]) : "v"(h), "v"(x0));
  asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r[1]) : "v"(h), "v"(x1));
  l = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, f16x2));
}

// Scale S_b of a body and the distances from its centre below which a target
// is near and above which it is far.  |K| 4 pi / k^3 <= (|aw| / k) t (sqrt(1 + t^2) + eta / k),
// t = 1 / (k r) (single layer: (|aw| / k) t eta / k).
struct MmBody {
  float S, near2;        // near: |D|^2 below this
  float kfar, kR, wk;    // far: k |D| above kfar; k R_b; S_b max |aw| / k
  float ek;              // eta / k
  int32_t e;             // log2 S_b
};
template <typename T>
__device__ __forceinline__ T mm_bound(int form, T wk, T t, T ek) {
  return wk * t * (form == 2 ? ek : sqrt((T)1 + t * t) + (form == 1 ? ek : (T)0));
}

__global__ __launch_bounds__(256) void mm_body_kernel(const BodyDev* __restrict__ bodies,
                                                      const float4* __restrict__ loc32,
                                                      const float4* __restrict__ aw32, int form,
                                                      MmBody* __restrict__ mb) {
  const BodyDev& B = bodies[blockIdx.x];
  float r2 = 0.0f, w2 = 0.0f;
  for (int i = threadIdx.x; i < B.n; i += 256) {
    const float4 a = aw32[B.off + i];
    r2 = fmaxf(r2, loc32[B.off + i].w);
    w2 = fmaxf(w2, a.x * a.x + a.y * a.y + a.z * a.z);
  }
  __shared__ float s0[256], s1[256];
  s0[threadIdx.x] = r2;
  s1[threadIdx.x] = w2;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
      s0[threadIdx.x] = fmaxf(s0[threadIdx.x], s0[threadIdx.x + h]);
      s1[threadIdx.x] = fmaxf(s1[threadIdx.x], s1[threadIdx.x + h]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double R = 1.0001 * sqrt((double)s0[0]), W = 1.0001 * sqrt((double)s1[0]), k = B.k;
    const double rho = 0.5 * R, ek = B.eta / k;
    const double lim = mm_bound(form, W / k, 1.0 / (k * rho), ek);
    double far = rho;                  // where the bound is below 2^-10 of that
    while (far < 1024.0 * rho && mm_bound(form, W / k, 1.0 / (k * far), ek) > 0x1p-10 * lim) far *= 2.0;
    int e = 0;
    (void)frexp(lim, &e);
    e = max(-120, min(120, 14 - e));
    MmBody M;
    M.S = (float)ldexp(1.0, e);
    M.near2 = (float)(1.0001 * (R + rho) * (R + rho));
    M.kfar = (float)(k * (R + far));
    M.kR = (float)(k * R);
    M.wk = (float)(W / k * ldexp(1.0, e));
    M.ek = (float)ek;
    M.e = e;
    mb[blockIdx.x] = M;
  }
}

// Source records: float4 pairs (y', c |y'|^2), S (aw / 2 c, aw . y') with y'
// the offset from the body centre and c = k^2 / MM_2PI (as the reciprocal FP32
// kernel stages them), and S eta |aw| / k^2.  Near targets cancel c |y'|^2 and
// aw . y' against the target's terms, so both are formed in FP64 from the other
// entries as rounded, and c with the FP32 2 pi that mm_eval takes it out with.
constexpr float MM_2PI = (float)TWO_PI;
__global__ void mm_records_kernel(const BodyDev* __restrict__ bodies, const int32_t* __restrict__ node_body,
                                  const float4* __restrict__ loc32, const float4* __restrict__ aw32,
                                  const float* __restrict__ ew32, const MmBody* __restrict__ mb, int64_t N,
                                  float4* __restrict__ rec, float* __restrict__ ewk) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int b = node_body[n];
  const double k = bodies[b].k;
  const double c = k * k / (double)MM_2PI;
  const float4 y = loc32[n], a = aw32[n];
  const float S = mb[b].S;
  const double yx = y.x, yy = y.y, yz = y.z, hw = 0.5 / c * S;
  const float wx = (float)(a.x * hw), wy = (float)(a.y * hw), wz = (float)(a.z * hw);
  rec[2 * n] = make_float4(y.x, y.y, y.z, (float)(c * fma(yx, yx, fma(yy, yy, yz * yz))));
  rec[2 * n + 1] = make_float4(wx, wy, wz, (float)(2.0 * c * fma(wx, yx, fma(wy, yy, wz * yz))));
  ewk[n] = ew32[n] * (float)(1.0 / (k * k)) * S;
}

// Largest |Re|, |Im| of mu per body and right-hand side, as the bits of a
// non-negative double (which order like the values; NaN above infinity).
// Workgroup: a body x two right-hand sides, in one launch; maxima met by atomics in
// cleared memory took two: 12 bodies of order 128, 2 right-hand sides, the whole sum
// 37.9 -> 34.7 us (the per-target kernel 36.8).  Eight right-hand sides a workgroup
// leave two bodies of order 8192 too few (33 right-hand sides 379 us against 364).
constexpr int MM_COLS = 2;
__global__ __launch_bounds__(1024) void mm_colmax_kernel(const BodyDev* __restrict__ bodies,
                                                         const double2* __restrict__ mu, int nrhs,
                                                         unsigned long long* __restrict__ colmax) {
  constexpr int COLS = MM_COLS, ROWS = 1024 / COLS;
  const int groups = (nrhs + COLS - 1) / COLS, body = blockIdx.x / groups;
  const int col = threadIdx.x % COLS, r = (int)(blockIdx.x % groups) * COLS + col;
  const int64_t off = bodies[body].off;
  const int n = bodies[body].n;
  unsigned long long m = 0;
  if (r < nrhs)
#pragma unroll 8
    for (int i = threadIdx.x / COLS; i < n; i += ROWS) {
      const double2 v = mu[(off + i) * nrhs + r];
      const unsigned long long x = __double_as_longlong(fabs(v.x)), y = __double_as_longlong(fabs(v.y));
      m = max(m, max(x, y));
    }
  for (int s = COLS; s < 64; s <<= 1) m = max(m, (unsigned long long)__shfl_xor((long long)m, s));
  __shared__ unsigned long long sm[16][COLS];
  if ((threadIdx.x & 63) < COLS) sm[threadIdx.x >> 6][col] = m;
  __syncthreads();
  if (threadIdx.x < COLS && r < nrhs) {
    for (int w = 1; w < 16; ++w) m = max(m, sm[w][col]);
    colmax[(int64_t)body * nrhs + r] = m;
  }
}

// log2 sigma of a body's column from its largest value (0 when that is zero or
// not finite)
__device__ __forceinline__ int mm_sigma(unsigned long long bits) {
  const double m = __longlong_as_double(bits);
  if (!(m > 0.0) || !(m <= 1.7e308)) return 0;
  int e = 0;
  (void)frexp(m, &e);
  return max(-780, min(15 - e, 780));
}

// log2 of what takes the sums over a body's sources out of the scales
__device__ __forceinline__ int mm_undo(const MmBody* __restrict__ mb, const unsigned long long* __restrict__ colmax,
                                       int body, int nrhs, int r) {
  return r < nrhs ? -(mm_sigma(colmax[(int64_t)body * nrhs + r]) + mb[body].e) : 0;
}

// Densities scaled, split and laid out as the B operands of the 32x32x16
// products, a group of right-hand sides r0 ... at a time: per half chunk of 16
// sources four fragments of 64 16-byte values, h, l of B1 and of B2.  A tile of 32
// right-hand sides (wide): B1 = Re mu, B2 = Im mu, one column each; a tile of
// 16: B1 = [Re mu | Im mu], B2 = [-Im mu | Re mu], 16 columns each.  Lane l of
// a fragment holds column l % 32 and the sources 8 (l / 32) ... + 7.
__global__ __launch_bounds__(256) void mm_pack_kernel(const double2* __restrict__ mu, int64_t halves, int nrhs,
                                                      int r0, int wide, int tiles,
                                                      const int32_t* __restrict__ node_body,
                                                      const unsigned long long* __restrict__ colmax,
                                                      u32x4* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int lane = (int)(t & 63);
  const int64_t hc = t >> 6;
  if (hc >= halves) return;
  const int col = lane & 31;
  const int tile = blockIdx.y;
  const bool second = !wide && col >= 16;
  const int r = r0 + tile * 32 + (wide ? col : (col & 15));
  const double2* v = mu + (hc * 16 + (lane >> 5) * 8) * nrhs + r;
  const int body = node_body[hc * 16];
  const double sc = r < nrhs ? ldexp(1.0, mm_sigma(colmax[(int64_t)body * nrhs + r])) : 0.0;
  float a[8], b[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const double2 m = r < nrhs ? v[(int64_t)s * nrhs] : make_double2(0.0, 0.0);
    const float re = (float)(m.x * sc), im = (float)(m.y * sc);
    a[s] = second ? im : re;
    b[s] = wide ? im : (second ? re : -im);
  }
  u32x4 fa[2], fb[2];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    uint32_t x, y;
    split2(a[2 * s], a[2 * s + 1], x, y);
    fa[0][s] = x; fa[1][s] = y;
    split2(b[2 * s], b[2 * s + 1], x, y);
    fb[0][s] = x; fb[1][s] = y;
  }
  u32x4* o = out + (tiles == 2 ? (hc >> 1) * 4 + tile * 2 + (hc & 1) : hc) * 4 * 64 + lane;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    o[q * 64] = fa[q];
    o[(2 + q) * 64] = fb[q];
  }
}

struct MmTarget {   // per target and source body (see the reciprocal FP32 kernel)
  float mx, my, mz, d2s, dns, ph0;
};

// The target at (x, y, z) against body B.  Returns how the wavefront's entries are
// scaled beyond S_b: -1 by their sizes (a target is near), 0 not at all, else by
// that power of two (all are far).
template <int FORM>
__device__ __forceinline__ int mm_target(const BodyDev& B, const MmBody& M, double x, double y, double z, double k,
                                          MmTarget& G) {
  const double c2 = 2.0 * k * k / (double)MM_2PI;
  const double Dx = B.cen[0] - x, Dy = B.cen[1] - y, Dz = B.cen[2] - z;
  const double D2 = fma(Dx, Dx, fma(Dy, Dy, Dz * Dz));
  const double Dn = sqrt(D2);
  double ph = k * Dn / TWO_PI;
  ph -= floor(ph);
  G.mx = (float)(c2 * Dx);
  G.my = (float)(c2 * Dy);
  G.mz = (float)(c2 * Dz);
  G.d2s = (float)(k * k * D2);
  // k |D| less what makes num over k r + k |D| revolutions of 2 pi again, not of
  // MM_2PI (r near |D|, where the phase difference counts)
  G.dns = (float)(k * Dn * (2.0 * TWO_PI / (double)MM_2PI - 1.0));
  G.ph0 = (float)ph;
  if (__any(!(D2 >= (double)M.near2))) return -1;
  if (!__all(G.dns > M.kfar)) return 0;
  float d = G.dns;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) d = fminf(d, __shfl_xor(d, o));
  int e = 0;
  (void)frexpf(mm_bound(FORM, M.wk, 1.0f / (d - M.kR), M.ek), &e);
  return __builtin_amdgcn_readfirstlane(max(0, min(14 - e, 100)));
}

// K (in units of k^3 / 4 pi, scaled by the records' S) of a target and the
// source with records Y, W, E.
template <int FORM>
__device__ __forceinline__ void mm_eval(const float4 Y, const float4 W, float E, const MmTarget& T, float& kr,
                                        float& ki) {
  const float num = fmaf(Y.x, T.mx, fmaf(Y.y, T.my, fmaf(Y.z, T.mz, Y.w)));
  const float r2s = fmaf(MM_2PI, num, T.d2s);
  const float irs = __builtin_amdgcn_rsqf(r2s);
  const float ph = fmaf(num, __builtin_amdgcn_rcpf(fmaf(r2s, irs, T.dns)), T.ph0);
  const float sn = __builtin_amdgcn_sinf(ph);
  const float cs = __builtin_amdgcn_cosf(ph);
  if constexpr (FORM == 2) {
    const float g = E * irs;
    kr = cs * g;
    ki = sn * g;
  } else {
    const float d = fmaf(W.x, T.mx, fmaf(W.y, T.my, fmaf(W.z, T.mz, W.w)));
    const float di = d * (irs * irs);
    kr = -(fmaf(cs, irs, sn) * di);
    ki = fmaf(-sn, irs, cs) * di;
    if constexpr (FORM == 1) {
      const float g = E * irs;
      kr = fmaf(g, sn, kr);
      ki = fmaf(-g, cs, ki);
    }
  }
}

// The A operands (h, l of Re K, h, l of Im K) of the lane's target and eight
// sources with records at R and E, scaled as mm_target says.  Near: entries beyond
// the bound of S_b scale the whole half chunk down; returns the power of two that undoes
// that (1 otherwise; entries that are not finite stay so).
template <int FORM>
__device__ __forceinline__ float mm_operands(const float4* R, const float* E, const MmTarget& G, int scaled,
                                             u32x4* f) {
  float kr[8], ki[8], undo = 1.0f;
#pragma unroll
  for (int s = 0; s < 8; ++s) mm_eval<FORM>(R[2 * s], R[2 * s + 1], E[FORM ? s : 0], G, kr[s], ki[s]);
  if (scaled > 0) {
    const float g = ldexpf(1.0f, scaled);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      kr[s] *= g;
      ki[s] *= g;
    }
  }
  if (scaled < 0) {
    float m = 0.0f;
#pragma unroll
    for (int s = 0; s < 8; ++s) m = fmaxf(m, fmaxf(fabsf(kr[s]), fabsf(ki[s])));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if (m >= 32768.0f && m < 3.0e38f) {
      int e = 0;
      (void)frexpf(m, &e);
      undo = ldexpf(1.0f, e - 14);
      const float g = ldexpf(1.0f, 14 - e);
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        kr[s] *= g;
        ki[s] *= g;
      }
    }
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    uint32_t x, y;
    split2(kr[2 * s], kr[2 * s + 1], x, y);
    f[0][s] = x; f[1][s] = y;
    split2(ki[2 * s], ki[2 * s + 1], x, y);
    f[2][s] = x; f[3][s] = y;
  }
  return undo;
}

__device__ __forceinline__ f32x16 mm_mma(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                0, 0);
}

// c += (a0 + a1)(b0 + b1) without a1 b1
__device__ __forceinline__ f32x16 mm_mma3(const u32x4* a, const u32x4* b, f32x16 c) {
  c = mm_mma(a[1], b[0], c);
  c = mm_mma(a[0], b[1], c);
  return mm_mma(a[0], b[0], c);
}

// The products of one half chunk (f: A operands, B operands at fb): a tile of
// 32 right-hand sides accumulates Re and Im apart, one of 16 [Re | Im].
template <int WIDE>
__device__ __forceinline__ void mm_products(u32x4* f, const u32x4* fb, f32x16* acc) {
  u32x4 b[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) b[q] = fb[q * 64];
  acc[0] = mm_mma3(f, b, acc[0]);
  if constexpr (WIDE) {
    acc[1] = mm_mma3(f, b + 2, acc[1]);
    acc[1] = mm_mma3(f + 2, b, acc[1]);
    f[2] ^= 0x80008000u;
    f[3] ^= 0x80008000u;
  }
  acc[0] = mm_mma3(f + 2, b + 2, acc[0]);
}

// FP32 sums of at most eight chunks (256 sources) of one body, added up in FP64
// times 2^e
template <int NA>
struct MmSums {
  f32x16 acc[NA];
  double sum[NA][16];
  int n, e;
  __device__ __forceinline__ void clear() {
    n = e = 0;
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        acc[a][i] = 0.0f;
        sum[a][i] = 0.0;
      }
  }
  __device__ __forceinline__ void flush(double f = 1.0) {
    f *= __hiloint2double((1023 + e) << 20, 0);   // 2^e
    n = 0;
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        sum[a][i] = fma((double)acc[a][i], f, sum[a][i]);
        acc[a][i] = 0.0f;
      }
  }
  // last: of its body, or of all
  __device__ __forceinline__ void end_chunk(bool last) {
    if (++n == 8 || last) flush();
  }
};

// No right-hand side of [r0, r1) is active in a lockstep solve: zeros for the
// nt targets from t0 on.
__device__ __forceinline__ bool mm_inactive(const int32_t* __restrict__ seg_active, int problem, int nrhs, int r0,
                                            int r1, int64_t t0, int nt, double2* __restrict__ dst) {
  if (!seg_active) return false;
  bool any = false;
  for (int r = r0; r < r1; ++r) any = any || seg_active[problem * nrhs + r] != 0;
  if (any) return false;
  const int nr = r1 - r0;
  for (int e = threadIdx.x; e < nt * nr; e += 256) dst[(t0 + e / nr) * nrhs + r0 + e % nr] = make_double2(0.0, 0.0);
  return true;
}

// The source chunks of a task: the body that holds every target is passed
// over; body and the end of its chunks follow the chunk number.
struct MmWalk {
  int own0 = 0, own1 = 0;   // chunks passed over
  int body = -1, end = 0;
  __device__ __forceinline__ MmWalk(const MmTask& T, const BodyDev* __restrict__ bodies) {
    if (T.body >= 0) {
      own0 = (int)(bodies[T.body].off / MM_C);
      own1 = own0 + bodies[T.body].n / MM_C;
    }
  }
  __device__ __forceinline__ int next(int c) const { return c >= own0 && c < own1 ? own1 : c; }
  __device__ __forceinline__ void start(int c, const BodyDev* __restrict__ bodies,
                                        const int32_t* __restrict__ node_body) {
    body = node_body[(int64_t)c * MM_C];
    end = (int)((bodies[body].off + bodies[body].n) / MM_C);
  }
  __device__ __forceinline__ void to(int c, const BodyDev* __restrict__ bodies) {
    while (c >= end) end += bodies[++body].n / MM_C;
  }
};

// Up to 32 (WIDE) or 16 right-hand sides from r0 on.  A workgroup takes 128
// targets, 32 per wavefront; the chunk's records and packed densities pass
// through LDS (double-buffered, the next chunk loaded meanwhile); lane l
// evaluates K for target l % 32 and the sources 8 (l / 32) ... + 7 of each
// half chunk, which is the A operand's layout, so K never leaves registers.
// Bound by vector issue (per pair 4 transcendentals at 8.3 cycles, 15 FP32 and
// 4 conversion instructions at 2.5 to 4.4, about 92 cycles per 64 pairs; 6 or
// 12 matrix instructions of 32 cycles per 512 pairs, which overlap little).
// 100 bodies of 2048 nodes (4.2e10 pairs): 16 right-hand sides 114.6 -> 36.4 ms,
// 32 202.6 -> 46.4 ms against the per-target kernel; register caps of 4 and 3
// wavefronts per SIMD are 4 % faster than 3 and 2 (8 % at 32, 46.4 and 50.4), except
// for the combined field with 32, whose larger evaluation spills at 3 (52.9 ms at
// 2, 56.9 at 3).  The targets' coordinates in LDS and the records four bytes a thread
// leave room for the scales of the sources' body (15 spilled registers and 47.3 ms
// without).  Bfloat16 in three parts (six
// products, nine vector instructions more per pair) took 51 and 73 ms; moving
// the products of one half chunk between the evaluations of the next gave nothing.
template <int WIDE, int FORM>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(WIDE ? FORM == 1 ? 2 : 3 : 4))) void pair_mmf_kernel(
    const MmTask* __restrict__ tasks, const BodyDev* __restrict__ bodies, const int32_t* __restrict__ node_body,
    const double* __restrict__ pos, int64_t N, const MmBody* __restrict__ mb, const u32x4* __restrict__ rec,
    const float* __restrict__ ewk, const u32x4* __restrict__ pack,
    const unsigned long long* __restrict__ colmax, int nrhs, int r0, const int32_t* __restrict__ seg_active,
    double2* __restrict__ partial) {
  constexpr int NV = 8 * 64;                     // packed 16-byte values per chunk
  constexpr int NA = 1 + WIDE;
  const MmTask T = tasks[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, half = lane >> 5;
  double2* dst = partial + (int64_t)T.slot * N * nrhs;
  if (mm_inactive(seg_active, T.problem, nrhs, r0, min(nrhs, r0 + 16 * NA), T.t0, T.nt, dst)) return;
  const int64_t tile0 = T.t0 + wave * 32;
  const bool live = wave * 32 < T.nt;
  __shared__ u32x4 sB[2][NV];
  __shared__ u32x4 sR[2][64];
  __shared__ float sE[2][FORM ? 32 : 1];
  const double k = T.k;
  __shared__ double sX[3][128];                  // the targets, read where the sources' body changes
  const int mybody = live ? node_body[tile0] : -1;
  const int64_t ti = live ? tile0 + col : T.t0;
  for (int d = half; d < 3; d += 2) sX[d][wave * 32 + col] = pos[d * N + ti];

  MmSums<NA> S;
  S.clear();
  MmTarget G;
  int scaled = 0, cur = -1, buf = 0;
  MmWalk W(T, bodies);
  u32x4 pre[2];
  uint32_t prec;                                 // records: four bytes per thread
  float pew = 0.0f;
  auto fetch = [&](int c) {
    const u32x4* p = pack + (int64_t)c * NV + tid;
#pragma unroll
    for (int q = 0; q < 2; ++q) pre[q] = p[q * 256];
    prec = ((const uint32_t*)rec)[(int64_t)c * 256 + tid];
    if (FORM && wave == 0) pew = ewk[(int64_t)c * MM_C + col];
  };
  int c = W.next(T.c0);
  if (c < T.c1) {
    fetch(c);
    W.start(c, bodies, node_body);
  }
  while (c < T.c1) {
#pragma unroll
    for (int q = 0; q < 2; ++q) sB[buf][tid + q * 256] = pre[q];
    ((uint32_t*)sR[buf])[tid] = prec;
    if (FORM && wave == 0) sE[buf][col] = pew;
    __syncthreads();
    const int cn = W.next(c + 1);
    if (cn < T.c1) fetch(cn);
    W.to(c, bodies);
    if (live && W.body != mybody) {
      if (W.body != cur) {
        cur = W.body;
        const int tc = wave * 32 + col;
        scaled = mm_target<FORM>(bodies[cur], mb[cur], sX[0][tc], sX[1][tc], sX[2][tc], k, G);
        S.e = mm_undo(mb, colmax, cur, nrhs, r0 + (WIDE ? col : (col & 15))) - max(scaled, 0);
      }
#pragma unroll
      for (int hc = 0; hc < 2; ++hc) {
        u32x4 f[4];
        const float undo = mm_operands<FORM>((const float4*)&sR[buf][(hc * 16 + half * 8) * 2],
                                             &sE[buf][FORM ? hc * 16 + half * 8 : 0], G, scaled, f);
        if (undo != 1.0f) S.flush();
        mm_products<WIDE>(f, &sB[buf][hc * 4 * 64 + lane], S.acc);
        if (undo != 1.0f) S.flush((double)undo);
      }
      S.end_chunk(cn >= min(W.end, T.c1));
    }
    buf ^= 1;
    c = cn;
  }
  if (!live) return;
  // element e of the lane: column l % 32, row 8 (e / 4) + 4 (l / 32) + e % 4
  const int r = r0 + (WIDE ? col : (col & 15));
  const double sc = k * k * k / FOUR_PI;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int64_t i = tile0 + 8 * (e >> 2) + 4 * half + (e & 3);
    const double im = WIDE ? S.sum[NA - 1][e] : __shfl_down(S.sum[0][e], 16);
    if ((WIDE || col < 16) && r < nrhs) dst[i * nrhs + r] = make_double2(S.sum[0][e] * sc, im * sc);
  }
}

// 33 to 64 right-hand sides from r0 on: two wavefronts share a tile of 32
// targets, each with 32 right-hand sides.  Each evaluates one half chunk of K
// for both (the operands pass through LDS) and multiplies the previous chunk,
// so every entry of K is evaluated once for all 64: 82 ms on the 100 bodies
// above, against 95 ms for two passes of the kernel above and 394 ms for the
// per-target kernel.
template <int FORM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void pair_mmf64_kernel(
    const MmTask* __restrict__ tasks, const BodyDev* __restrict__ bodies, const int32_t* __restrict__ node_body,
    const double* __restrict__ pos, int64_t N, const MmBody* __restrict__ mb, const u32x4* __restrict__ rec,
    const float* __restrict__ ewk, const u32x4* __restrict__ pack,
    const unsigned long long* __restrict__ colmax, int nrhs, int r0, const int32_t* __restrict__ seg_active,
    double2* __restrict__ partial) {
  constexpr int NV = 16 * 64;                    // packed 16-byte values per chunk
  const MmTask T = tasks[blockIdx.x >> 1];
  const int sub = (blockIdx.x & 1) * 64;         // this workgroup's half of the task's targets
  const int nt = min(64, T.nt - sub);
  if (nt <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tile = wave >> 1, hw = wave & 1;     // the wavefront's tile; its half chunk and right-hand sides
  const int col = lane & 31, half = lane >> 5;
  double2* dst = partial + (int64_t)T.slot * N * nrhs;
  if (mm_inactive(seg_active, T.problem, nrhs, r0, min(nrhs, r0 + 64), T.t0 + sub, nt, dst)) return;
  const int64_t tile0 = T.t0 + sub + tile * 32;
  const bool live = tile * 32 < nt;
  __shared__ u32x4 sB[2][NV];
  __shared__ u32x4 sA[2][2][2][4 * 64];          // buffer, tile, half chunk
  __shared__ u32x4 sR[2][64];
  __shared__ float sE[2][FORM ? 32 : 1];
  __shared__ float sU[2][2][2];                  // what undoes the half chunk's scaling
  const double k = T.k;
  const int mybody = live ? node_body[tile0] : -1;
  const int64_t ti = live ? tile0 + col : T.t0;
  __shared__ double sX[3][64];                   // the targets, read where the sources' body changes
  const int tc = tile * 32 + col;
  for (int d = half; d < 3; d += 2) sX[d][tc] = pos[d * N + ti];
  const int r = r0 + hw * 32 + col;              // the lane's right-hand side

  MmSums<2> S;
  S.clear();
  MmTarget G;
  int how = 0;                                   // mm_target's scaling of the body evaluated
  int cur = -1, summed = -1;                     // bodies evaluated, multiplied
  MmWalk W(T, bodies);
  u32x4 preB[4];
  uint32_t preR;                                 // records: four bytes per thread
  float preE = 0.0f;
  auto fetch_b = [&](int c) {
    if (c >= T.c1) return;
    const u32x4* p = pack + (int64_t)c * NV + tid;
#pragma unroll
    for (int q = 0; q < 4; ++q) preB[q] = p[q * 256];
  };
  auto fetch_r = [&](int c) {
    if (c >= T.c1) return;
    preR = ((const uint32_t*)rec)[(int64_t)c * 256 + tid];
    if (FORM && wave == 0) preE = ewk[(int64_t)c * MM_C + col];
  };
  auto store_b = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 4; ++q) sB[buf][tid + q * 256] = preB[q];
  };
  auto store_r = [&](int buf) {
    ((uint32_t*)sR[buf])[tid] = preR;
    if (FORM && wave == 0) sE[buf][col] = preE;
  };
  // whether the tile meets the chunk W is at (G, how and scales set for it)
  int scales = 0;
  auto meets = [&]() {
    if (!live || W.body == mybody) return false;
    if (W.body != cur) {
      cur = W.body;
      how = mm_target<FORM>(bodies[cur], mb[cur], sX[0][tc], sX[1][tc], sX[2][tc], k, G);
      scales = mm_undo(mb, colmax, cur, nrhs, r) - max(how, 0);
    }
    return true;
  };
  // K of the wavefront's half chunk, from record buffer rb to operand buffer ab
  auto evaluate = [&](int rb, int ab, int scaled) {
    u32x4 f[4];
    const float undo = mm_operands<FORM>((const float4*)&sR[rb][(hw * 16 + half * 8) * 2],
                                         &sE[rb][FORM ? hw * 16 + half * 8 : 0], G, scaled, f);
    if (scaled < 0 && lane == 0) sU[ab][tile][hw] = undo;
    u32x4* o = &sA[ab][tile][hw][lane];
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q * 64] = f[q];
  };
  auto multiply = [&](int ab, int hc) {
    u32x4 f[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) f[q] = sA[ab][tile][hc][q * 64 + lane];
    mm_products<1>(f, &sB[ab][(hw * 2 + hc) * 4 * 64 + lane], S.acc);
  };

  // in step i, after its barrier: chunk i is multiplied, chunk i + 1 evaluated,
  // and the densities of i + 1 and the records of i + 2 stored into the buffers
  // that step i - 1 was the last to read
  int c0 = W.next(T.c0), c1 = W.next(c0 + 1), c2 = W.next(c1 + 1);
  bool use = false;   // chunk i
  int scaled = 0;
  if (c0 < T.c1) {
    fetch_b(c0);
    fetch_r(c0);
    store_b(0);
    store_r(0);
    fetch_r(c1);
    if (c1 < T.c1) store_r(1);
    fetch_b(c1);
    fetch_r(c2);
    __syncthreads();
    W.start(c0, bodies, node_body);
    use = meets();
    scaled = how;
    if (use) evaluate(0, 0, scaled);
    S.e = scales;
    summed = cur;
  }
  for (int i = 0; c0 < T.c1; ++i) {
    __syncthreads();
    const int p0 = i & 1, p1 = p0 ^ 1;
    if (c1 < T.c1) store_b(p1);
    if (c2 < T.c1) store_r(p0);
    const int c3 = W.next(c2 + 1);
    fetch_b(c2);
    fetch_r(c3);
    bool use1 = false;
    if (c1 < T.c1) {
      W.to(c1, bodies);
      use1 = meets();
    }
    if (use && use1 && scaled >= 0 && how == 0) {
      // no branch between the two products and the evaluation: 5 % faster
      multiply(p0, 0);
      evaluate(p1, p1, 0);
      multiply(p0, 1);
    } else {
      if (use1) evaluate(p1, p1, how);
      if (use) {
#pragma unroll 1
        for (int hc = 0; hc < 2; ++hc) {
          const float undo = scaled < 0 ? sU[p0][tile][hc] : 1.0f;
          if (undo != 1.0f) S.flush();
          multiply(p0, hc);
          if (undo != 1.0f) S.flush((double)undo);
        }
      }
    }
    S.end_chunk(summed != cur || c1 >= T.c1);
    S.e = scales;
    summed = cur;
    use = use1;
    scaled = how;
    c0 = c1;
    c1 = c2;
    c2 = c3;
  }
  if (!live || r >= nrhs) return;
  const double sc = k * k * k / FOUR_PI;
  // element e of the lane: column l % 32, row 8 (e / 4) + 4 (l / 32) + e % 4
#pragma unroll
  for (int e = 0; e < 16; ++e)
    dst[(tile0 + 8 * (e >> 2) + 4 * half + (e & 3)) * nrhs + r] =
        make_double2(S.sum[0][e] * sc, S.sum[1][e] * sc);
}

// ---------------------------------------------------------------- FP64 path
// The same scheme on v_mfma_f64_16x16x4f64, for pair sums (tasks given; the
// targets' own body is left out), for evaluation points off the surfaces and
// for far-field directions (tasks null: 128 targets x one of gridDim.y ranges
// of a problem's sources x problem).  Lane l evaluates K for targets l % 16 of
// two tiles and source l / 16 of each step of four, which is the A operand's
// layout; a tile of 8 right-hand sides has columns [Re mu | Im mu] against
// Re K and [-Im mu | Re mu] against Im K.
// Pair sums and points: with t = 1 / (k r), K = k e^{ikr} (i - t) aw.(y - x) / r^2 / 4 pi
// (combined field: minus i eta |aw| e^{ikr} / r; single layer: |aw| e^{ikr} / r),
// the sine and cosine from a table of k sin, k cos.  Directions xhat: K = (-i k xhat.aw) e^{-i k xhat.y}
// (combined field: plus -i eta |aw| e^{...}; single layer: |aw| e^{...}) / 4 pi.
typedef double f64x4 __attribute__((ext_vector_type(4)));

enum { MM_DOUBLE = 0, MM_COMBINED = 1, MM_SINGLE = 2, MM_FAR = 3 };   // far field: MM_FAR + formulation

struct MmTargets {        // coordinate c of target i: x[i step + c stride]
  const double* x;
  int64_t step, stride;
  int64_t count;          // targets
  const int2* items;      // far field: paired directions (item: direction, its exact negation), or null
  int64_t n_items;        // items, or targets without a list
  const int64_t* pinfo;   // first node of every problem, the end of the last, then their k (as bits)
  int32_t nprob, prob0;   // problems in pinfo, first problem evaluated (gridDim.z of them)
};

// VEC: up to VEC right-hand sides by vector fmas instead (each lane adds up its
// targets over every fourth source, the four sums are added at the end).
// PAIRS (far field): the lane's two targets are a direction and its negation,
// with one sine and cosine for both.
// Bound by FP64 issue: about 40 instructions a pair for K (4.4 cycles each, 200
// per 64 pairs with the table reads), 145 cycles of matrix time per tile of 8
// right-hand sides, or 25 of vector time each.  40 bodies of 2048 nodes (6.5e9
// pairs), against the per-target kernel: 2 right-hand sides 17.4 -> 11.0 ms,
// 4 17.8 -> 13.4 (14.2 on the matrix cores), 8 21.4 -> 14.2, 16 41.8 -> 20.2, 32 81.3 -> 32.3.
// Far field of 57,600 nodes in 40,000 directions 3.1 -> 2.4 ms (28.7 vector
// instructions a pair, the vector ALUs 90 % busy at the 1.84 GHz that FP64 work
// leaves; before, nine LDS reads a pair for one direction per lane).
template <int NT, int VEC, int FORM, bool PAIRS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NT > 2 ? 2 : 3))) void mm_sum_kernel(
    const MmTask* __restrict__ tasks, MmTargets P, const BodyDev* __restrict__ bodies,
    const int32_t* __restrict__ node_body, const double* __restrict__ pos, const double* __restrict__ aw,
    const double* __restrict__ ew, int64_t N, const double2* __restrict__ mu, int nrhs, int r0,
    const int32_t* __restrict__ seg_active, double2* __restrict__ partial) {
  constexpr bool FAR = FORM >= MM_FAR;
  constexpr bool EW = FORM % 3 != MM_DOUBLE;     // the single-layer weights enter
  constexpr int NM = VEC ? 1 : NT;               // groups of 8 right-hand sides staged
  constexpr int PER = PAIRS ? 16 : 32;           // items per wavefront
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 15, kq = lane >> 4;
  MmTask T;
  int64_t slot = 0;
  if (tasks) {
    T = tasks[blockIdx.x];
    slot = T.slot;
  } else {
    const int pr = P.prob0 + blockIdx.z;
    const int32_t q0 = (int32_t)(P.pinfo[pr] / MM_C), q1 = (int32_t)(P.pinfo[pr + 1] / MM_C);
    T.t0 = (int64_t)blockIdx.x * (4 * PER);
    T.nt = (int32_t)min((int64_t)(4 * PER), P.n_items - T.t0);
    T.c0 = q0 + (int32_t)((int64_t)(q1 - q0) * blockIdx.y / gridDim.y);
    T.c1 = q0 + (int32_t)((int64_t)(q1 - q0) * (blockIdx.y + 1) / gridDim.y);
    T.body = -1;
    T.problem = pr;
    T.k = __longlong_as_double(P.pinfo[P.nprob + 1 + pr]);
    slot = (int64_t)blockIdx.y * gridDim.z + blockIdx.z;
  }
  double2* dst = partial + slot * P.count * nrhs;
  if (mm_inactive(seg_active, T.problem, nrhs, r0, min(nrhs, r0 + 8 * NM), T.t0, T.nt, dst)) return;
  const double k = T.k;
  const int64_t item0 = T.t0 + wave * PER;
  const bool live = wave * PER < T.nt;
  const int mybody = tasks && live ? node_body[item0] : -1;
  // target of the tile's row q (16 rows), and whether there is one
  auto target = [&](int t, int q, int64_t* i) {
    const int64_t m = item0 + (PAIRS ? q : 16 * t + q);
    const bool ok = m < P.n_items;
    *i = ok ? m : P.n_items - 1;
    if (FAR && P.items) *i = PAIRS && t ? P.items[*i].y : P.items[*i].x;
    return ok;
  };
  double tx[2], ty[2], tz[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    int64_t i;
    (void)target(t, col, &i);
    tx[t] = P.x[i * P.step];
    ty[t] = P.x[i * P.step + P.stride];
    tz[t] = P.x[i * P.step + 2 * P.stride];
  }
  __shared__ double2 sQ[2][3][MM_C];             // (x, y), (z, awx), (awy, awz)
  __shared__ double sE[2][EW ? MM_C : 1];        // ew (ew / k)
  __shared__ double2 sM[2][NM][MM_C][8];
  __shared__ double2 sTab[512];
  fill_tab512(sTab, tid, 256, FAR ? 1.0 : k);    // ordered by the first chunk's barrier

  f64x4 acc[2][NT ? NT : 1];
  double vr[2][VEC ? VEC : 1], vi[2][VEC ? VEC : 1];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[t][n] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < VEC; ++r) vr[t][r] = vi[t][r] = 0.0;
  }
  const double u512 = U512;                      // phases in 512ths of a revolution
  const double ku = (FAR ? -k : k) * u512;       // far field: the phase -k xhat.y
  // what ku leaves of k 512 / 2 pi (without it every phase is off by the same
  // 2^-54 of itself, which does not average out over the sources)
  const double kul = fma(k, u512, -ku) + k * U512_LOW;
  const double ik = FAR ? 0.0 : 1.0 / k;
  double X[2], Y[2], Z[2];                       // far field: k xhat, and ku xhat in tx, ty, tz
  if (FAR) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      X[t] = k * tx[t];
      Y[t] = k * ty[t];
      Z[t] = k * tz[t];
      tx[t] *= ku;
      ty[t] *= ku;
      tz[t] *= ku;
    }
  }
  int buf = 0;
  MmWalk W(T, bodies);
  double2 preM[NM];
  double2 preQ[3];
  double preE = 0.0;
  // thread tid loads right-hand side tid % 8 of source tid / 8; threads 0-31 also the records
  auto fetch = [&](int c) {
    const int64_t j = (int64_t)c * MM_C + (tid >> 3);
#pragma unroll
    for (int n = 0; n < NM; ++n) {
      const int r = r0 + 8 * n + (tid & 7);
      preM[n] = r < nrhs ? mu[j * nrhs + r] : make_double2(0.0, 0.0);
    }
    if (tid < MM_C) {
      const int64_t i = (int64_t)c * MM_C + tid;
      preQ[0] = make_double2(pos[i], pos[N + i]);
      preQ[1] = make_double2(pos[2 * N + i], aw[i]);
      preQ[2] = make_double2(aw[N + i], aw[2 * N + i]);
      if (EW) preE = FAR ? ew[i] : ew[i] / k;
    }
  };
  int c = W.next(T.c0);
  if (c < T.c1) {
    fetch(c);
    if (tasks) W.start(c, bodies, node_body);
  }
  const uint32_t flip = col < 8 ? 0x80000000u : 0u;   // sign of the second operand's columns
  while (c < T.c1) {
    if (tasks) W.to(c, bodies);
#pragma unroll
    for (int n = 0; n < NM; ++n) sM[buf][n][tid >> 3][tid & 7] = preM[n];
    if (tid < MM_C) {
#pragma unroll
      for (int q = 0; q < 3; ++q) sQ[buf][q][tid] = preQ[q];
      if (EW) sE[buf][tid] = preE;
    }
    __syncthreads();
    const int cn = W.next(c + 1);
    if (cn < T.c1) fetch(cn);
    if (live && (!tasks || W.body != mybody)) {
#pragma unroll 2
      for (int st = 0; st < MM_C / 4; ++st) {
        const int j = 4 * st + kq;
        const double2 q0 = sQ[buf][0][j], q1 = sQ[buf][1][j], q2 = sQ[buf][2][j];
        const double e = EW ? sE[buf][j] : 0.0;
        double kr[2], ki[2], sn = 0.0, cs = 0.0, d = 0.0;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          if constexpr (FAR) {
            // the negated direction: d and the sine change sign
            if (PAIRS && t) {
              sn = -sn;
              d = -d;
            } else {
              sincos_tab512(fma(tx[t], q0.x, fma(ty[t], q0.y, tz[t] * q1.x)), sTab, &sn, &cs);
              d = fma(X[t], q1.y, fma(Y[t], q2.x, Z[t] * q2.y));
            }
            if constexpr (FORM == MM_FAR + MM_SINGLE) {
              kr[t] = e * cs;
              ki[t] = e * sn;
            } else {
              const double a = EW ? d + e : d;
              kr[t] = a * sn;
              ki[t] = -(a * cs);
            }
          } else {
            const double dx = q0.x - tx[t], dy = q0.y - ty[t], dz = q1.x - tz[t];
            const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
            const double ir = rsqrt_pos(r2);
            sincos_tab512_scaled(r2 * ir, ku, kul, sTab, &sn, &cs);
            if constexpr (FORM == MM_SINGLE) {
              const double g = e * ir;
              kr[t] = cs * g;
              ki[t] = sn * g;
            } else {
              d = fma(q1.y, dx, fma(q2.x, dy, q2.y * dz)) * (ir * ir);
              const double it = ir * ik;
              kr[t] = -(fma(cs, it, sn) * d);
              ki[t] = fma(-sn, it, cs) * d;
              if constexpr (FORM == MM_COMBINED) {
                const double g = e * ir;
                kr[t] = fma(g, sn, kr[t]);
                ki[t] = fma(-g, cs, ki[t]);
              }
            }
          }
        }
        if constexpr (VEC != 0) {
#pragma unroll
          for (int r = 0; r < VEC; ++r) {
            const double2 m = sM[buf][0][j][r];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              vr[t][r] = fma(kr[t], m.x, fma(-ki[t], m.y, vr[t][r]));
              vi[t][r] = fma(kr[t], m.y, fma(ki[t], m.x, vi[t][r]));
            }
          }
        } else {
          double b1[NT ? NT : 1], b2[NT ? NT : 1];
#pragma unroll
          for (int n = 0; n < NT; ++n) {
            const double* m = (const double*)&sM[buf][n][j][col & 7];
            b1[n] = m[col >> 3];
            const double x = m[1 - (col >> 3)];
            b2[n] = __hiloint2double(__double2hiint(x) ^ flip, __double2loint(x));
          }
#pragma unroll
          for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int t = 0; t < 2; ++t)
              acc[t][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(kr[t], b1[n], acc[t][n], 0, 0, 0);
#pragma unroll
          for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int t = 0; t < 2; ++t)
              acc[t][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(ki[t], b2[n], acc[t][n], 0, 0, 0);
        }
      }
    }
    buf ^= 1;
    c = cn;
  }
  if (!live) return;
  const double sc = 1.0 / FOUR_PI;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    int64_t i;
    if constexpr (VEC != 0) {
      const bool ok = target(t, col, &i) && kq == 0;
#pragma unroll
      for (int r = 0; r < VEC; ++r) {
        double re = vr[t][r], im = vi[t][r];
        re += __shfl_xor(re, 16);
        im += __shfl_xor(im, 16);
        re += __shfl_xor(re, 32);
        im += __shfl_xor(im, 32);
        if (ok && r0 + r < nrhs) dst[i * nrhs + r0 + r] = make_double2(re * sc, im * sc);
      }
    } else {
      // element e of the lane: column l % 16, row l / 16 + 4 e of the tile
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool ok = target(t, kq + 4 * e, &i) && col < 8;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          const double re = acc[t][n][e], im = __shfl_down(re, 8);
          const int r = r0 + 8 * n + col;
          if (ok && r < nrhs) dst[i * nrhs + r] = make_double2(re * sc, im * sc);
        }
      }
    }
  }
}

// ---------------------------------------------------------------- plan and launch
static size_t align256(size_t b) { return (b + 255) / 256 * 256; }

// Target blocks of MM_T nodes of one problem, each against `slots` ranges of
// the problem's source chunks, sorted by decreasing cost: at least 24
// workgroups per compute unit (about eight rounds of those the chip holds; with
// four rounds the last one cost 6 % on the 100 bodies above, with more nothing
// was gained), at least eight chunks each (the sums' FP64 step).  Sums too small
// for a workgroup per compute unit that way are split further, down to single
// chunks: 5 bodies of order 96, FP64, 2 right-hand sides 51.1 -> 22.1 us, 64
// 188 -> 39.8 (FP32 51.0 -> 31.9, 49.2 -> 34.3); 12 of order 128 37.2 -> 28.9 and
// 116 -> 72.3 (41.3 -> 37.9, 44.6 -> 47.6).  Up to two workgroups per compute unit
// the 12 take 30.6 and 74.1 us (38.3, 53.2).
static void plan_mm(qax_problem* p, int cu_count, std::vector<MmTask>& tasks) {
  auto& M = p->mm;
  int64_t tblocks = 0, cmax = 0;
  for (int pr = 0; pr < p->n_problems; ++pr) {
    const int64_t n = p->off[p->prob_body0[pr + 1]] - p->off[p->prob_body0[pr]];
    tblocks += (n + MM_T - 1) / MM_T;
    if (p->prob_body0[pr + 1] - p->prob_body0[pr] > 1) cmax = std::max(cmax, n / MM_C);   // no pairs in one body
  }
  tblocks = std::max<int64_t>(tblocks, 1);
  const int64_t full = std::min<int64_t>((24LL * cu_count + tblocks - 1) / tblocks, cmax / 8);
  const int64_t small = std::min<int64_t>(cu_count / tblocks, cmax);
  const int64_t slots = std::max<int64_t>(1, std::min<int64_t>(32, std::max(full, small)));
  M.slots = (int)slots;
  // the body that holds every target of a block, or -1
  std::vector<int32_t> body;
  body.reserve(tblocks);
  // a problem's tasks take at most four costs (whole and last blocks, source
  // ranges a chunk apart): listed class by class
  struct Class { int64_t cost, block0; int32_t pr; bool last, longer; };
  std::vector<Class> classes;
  for (int pr = 0; pr < p->n_problems; ++pr) {
    const int b0 = (int)p->prob_body0[pr], b1 = (int)p->prob_body0[pr + 1];
    const int64_t n0 = p->off[b0], n1 = p->off[b1], q = (n1 - n0) / MM_C / slots;
    const int64_t block0 = (int64_t)body.size();
    int lo = b0;
    for (int64_t t0 = n0; t0 < n1; t0 += MM_T) {
      while (lo + 1 < b1 && p->off[lo + 1] <= t0) ++lo;
      body.push_back(p->off[lo + 1] >= std::min<int64_t>(t0 + MM_T, n1) ? lo : -1);
    }
    for (int last = 0; last < 2; ++last)
      for (int longer = 0; longer < 2; ++longer)
        classes.push_back(Class{(last ? (n1 - n0) % MM_T : MM_T) * (q + longer), block0, pr, last != 0, longer != 0});
  }
  std::stable_sort(classes.begin(), classes.end(), [](const Class& a, const Class& b) { return a.cost > b.cost; });
  tasks.clear();
  tasks.reserve((size_t)(tblocks * slots));
  for (const Class& C : classes) {
    const int64_t n0 = p->off[p->prob_body0[C.pr]], n1 = p->off[p->prob_body0[C.pr + 1]];
    const int64_t c0 = n0 / MM_C, nc = (n1 - n0) / MM_C, whole = (n1 - n0) / MM_T;
    const int64_t end = C.last ? (n1 - n0 + MM_T - 1) / MM_T : whole;
    for (int64_t b = C.last ? whole : 0; b < end; ++b)
      for (int s = 0; s < slots; ++s) {
        MmTask T;
        T.t0 = n0 + b * MM_T;
        T.nt = (int32_t)std::min<int64_t>(MM_T, n1 - T.t0);
        T.c0 = (int32_t)(c0 + nc * s / slots);
        T.c1 = (int32_t)(c0 + nc * (s + 1) / slots);
        T.slot = s;
        T.body = body[C.block0 + b];
        T.problem = C.pr;
        T.k = p->k[C.pr];
        if ((T.c1 - T.c0 > nc / slots) == C.longer) tasks.push_back(T);
      }
  }
}

// Made on first use (not inside a capture; nothing here waits): the task table, a
// function of the node ranges and wavenumbers, which a rebuild that keeps them
// keeps too, and for FP32 the bodies' scales and source records, functions of the
// geometry and the formulation.  First call after a build, above the next ones:
// N = 5120 44 us and N = 44,800 128 with both made, sorted and waited for each
// time; 3 to 15 now with the table kept, 18 to 54 with another.
hipError_t ensure_mm_plan(qax_problem* p, int prec, int cu_count) {
  auto& M = p->mm;
  hipError_t e = hipSuccess;
  if (!M.d_tasks) {
    plan_mm(p, cu_count, M.tasks);
    if ((e = dev_alloc(p, (void**)&M.d_tasks, sizeof(MmTask) * M.tasks.size())) != hipSuccess) return e;
    e = hipMemcpyAsync(M.d_tasks, M.tasks.data(), sizeof(MmTask) * M.tasks.size(), hipMemcpyHostToDevice, p->stream);
    if (e != hipSuccess) {
      free_mm_tasks(p);
      return e;
    }
    ++p->generation;
  }
  if (prec == QAX_FP64 || M.d_mem) return hipSuccess;
  const size_t bb = align256(sizeof(MmBody) * p->n_bodies), br = align256((size_t)p->N * 32);
  if ((e = dev_alloc(p, &M.d_mem, bb + br + (size_t)p->N * 4)) != hipSuccess) return e;
  char* m = (char*)M.d_mem;
  M.d_bodies = m;
  M.d_rec = m + bb;
  M.d_ewk = (float*)(m + bb + br);
  hipLaunchKernelGGL(mm_body_kernel, dim3((unsigned)p->n_bodies), dim3(256), 0, p->stream, p->d_bodies,
                     (const float4*)p->d_loc32, (const float4*)p->d_aw32, p->form(), (MmBody*)M.d_bodies);
  hipLaunchKernelGGL(mm_records_kernel, dim3((unsigned)((p->N + 255) / 256)), dim3(256), 0, p->stream, p->d_bodies,
                     p->d_node_body, (const float4*)p->d_loc32, (const float4*)p->d_aw32, p->d_ew32,
                     (const MmBody*)M.d_bodies, p->N, (float4*)M.d_rec, M.d_ewk);
  e = hipGetLastError();
  if (e != hipSuccess) free_mm_records(p);
  ++p->generation;
  return e;
}

// after a change of the geometry or formulation
void free_mm_records(qax_problem* p) {
  dev_release(p, p->mm.d_mem);
  p->mm.d_mem = nullptr;
}

// after a change of the node ranges or wavenumbers
void free_mm_tasks(qax_problem* p) {
  dev_release(p, p->mm.d_tasks);
  p->mm.d_tasks = nullptr;
  p->mm.tasks.clear();
}

static size_t mm_pack_values(const qax_problem* p, int nrhs) {
  return (size_t)(p->N / MM_C) * (nrhs > 32 ? 16 : 8) * 64;
}

size_t mm_work_bytes(const qax_problem* p, int prec, int nrhs) {
  size_t b = align256((size_t)p->mm.slots * p->N * nrhs * 16);
  if (prec != QAX_FP64)
    b += align256((size_t)p->n_bodies * nrhs * 8) + mm_pack_values(p, nrhs) * sizeof(u32x4);
  return b;
}

// Partial sums of the FP32 pair sum (slots x N x nrhs at `work`).
hipError_t launch_pair_mmf(qax_problem* p, const double* mu, int nrhs, double* work) {
  char* m = (char*)work;
  auto take = [&](size_t bytes) {
    char* q = m;
    m += align256(bytes);
    return q;
  };
  double2* partial = (double2*)take((size_t)p->mm.slots * p->N * nrhs * 16);
  const MmBody* mb = (const MmBody*)p->mm.d_bodies;
  unsigned long long* colmax = (unsigned long long*)take((size_t)p->n_bodies * nrhs * 8);
  u32x4* pack = (u32x4*)m;
  const int form = p->form();
  const hipStream_t s = p->stream;
  const int64_t halves = p->N / 16;
  const unsigned groups = (unsigned)((nrhs + MM_COLS - 1) / MM_COLS);
  hipLaunchKernelGGL(mm_colmax_kernel, dim3((unsigned)p->n_bodies * groups), dim3(1024), 0, s, p->d_bodies,
                     (const double2*)mu, nrhs, colmax);
  for (int r0 = 0; r0 < nrhs; r0 += 64) {
    const int left = nrhs - r0, wide = left > 16, tiles = left > 32 ? 2 : 1;
    hipLaunchKernelGGL(mm_pack_kernel, dim3((unsigned)((halves * 64 + 255) / 256), (unsigned)tiles), dim3(256), 0, s,
                       (const double2*)mu, halves, nrhs, r0, wide, tiles, p->d_node_body, colmax, pack);
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3((unsigned)(p->mm.tasks.size() * tiles)), dim3(256), 0, s, p->mm.d_tasks,
                         p->d_bodies, p->d_node_body, p->d_pos, p->N, mb, (const u32x4*)p->mm.d_rec, p->mm.d_ewk,
                         pack, colmax, nrhs, r0, p->seg_active, partial);
    };
    if (tiles == 2) go(form == 1 ? pair_mmf64_kernel<1> : form == 2 ? pair_mmf64_kernel<2> : pair_mmf64_kernel<0>);
    else if (wide) go(form == 1 ? pair_mmf_kernel<1, 1> : form == 2 ? pair_mmf_kernel<1, 2> : pair_mmf_kernel<1, 0>);
    else go(form == 1 ? pair_mmf_kernel<0, 1> : form == 2 ? pair_mmf_kernel<0, 2> : pair_mmf_kernel<0, 0>);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int V>
using I = std::integral_constant<int, V>;

// FP64 sums over the pair-sum tasks or other targets, right-hand sides 32 at a time.
template <int FORM, bool PAIRS>
static hipError_t launch_mm_sum(qax_problem* p, const MmTask* tasks, const MmTargets& P, dim3 grid, const double* mu,
                                int nrhs, double* partial) {
  for (int r0 = 0; r0 < nrhs; r0 += 32) {
    auto go = [&](auto nt, auto vec) {
      hipLaunchKernelGGL((mm_sum_kernel<decltype(nt)::value, decltype(vec)::value, FORM, PAIRS>), grid, dim3(256), 0,
                         p->stream, tasks, P, p->d_bodies, p->d_node_body, p->d_pos, p->d_aw, p->d_ew, p->N,
                         (const double2*)mu, nrhs, r0, p->seg_active, (double2*)partial);
    };
    const int left = nrhs - r0;
    if (left == 1) go(I<0>{}, I<1>{});
    else if (left == 2) go(I<0>{}, I<2>{});
    else if (left <= 4) go(I<0>{}, I<4>{});
    else if (left <= 8) go(I<1>{}, I<0>{});
    else if (left <= 16) go(I<2>{}, I<0>{});
    else if (left <= 24) go(I<3>{}, I<0>{});
    else go(I<4>{}, I<0>{});
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int BASE, bool PAIRS>
static hipError_t launch_mm_forms(qax_problem* p, const MmTask* tasks, const MmTargets& P, dim3 grid,
                                  const double* mu, int nrhs, double* partial) {
  switch (p->form()) {
    case 1: return launch_mm_sum<BASE + MM_COMBINED, PAIRS>(p, tasks, P, grid, mu, nrhs, partial);
    case 2: return launch_mm_sum<BASE + MM_SINGLE, PAIRS>(p, tasks, P, grid, mu, nrhs, partial);
    default: return launch_mm_sum<BASE + MM_DOUBLE, PAIRS>(p, tasks, P, grid, mu, nrhs, partial);
  }
}

// Partial sums of the FP64 pair sum (slots x N x nrhs at `work`).
hipError_t launch_pair_mmd(qax_problem* p, const double* mu, int nrhs, double* work) {
  const MmTargets P = {p->d_pos, 1, p->N, p->N, nullptr, p->N, nullptr, 0, 0};
  return launch_mm_forms<MM_DOUBLE, false>(p, p->mm.d_tasks, P, dim3((unsigned)p->mm.tasks.size()), mu, nrhs, work);
}

// Ranges of the sources for `count` targets of `nprob` problems from prob0 on:
// 24 workgroups per compute unit as for the pair sums, at least two chunks each
// (single chunks where that leaves compute units idle: 100 directions of 12 bodies
// of order 128 34.5 us against 30.7).
int mm_slots(const qax_problem* p, int64_t count, int prob0, int nprob, int cu_count) {
  int64_t cmax = 1;
  for (int pr = prob0; pr < prob0 + nprob; ++pr)
    cmax = std::max(cmax, (p->off[p->prob_body0[pr + 1]] - p->off[p->prob_body0[pr]]) / MM_C);
  const int64_t blocks = (count + MM_T - 1) / MM_T * nprob;
  return (int)std::max<int64_t>(1, std::min<int64_t>({64, cmax / 2, (24LL * cu_count + blocks - 1) / blocks}));
}

// Near field of one problem at M points (SoA); partial: slots x M x nrhs.
hipError_t launch_mm_near(qax_problem* p, const double* mu, int nrhs, const double* pts, int64_t M, int problem,
                          int slots, double* partial) {
  const MmTargets P = {pts, 1, M, M, nullptr, M, p->d_pinfo, p->n_problems, problem};
  return launch_mm_forms<MM_DOUBLE, false>(p, nullptr, P, dim3((unsigned)((M + MM_T - 1) / MM_T), (unsigned)slots), mu,
                                           nrhs, partial);
}

// Far field of every problem in M directions (AoS); partial: slots x problems x
// M x nrhs.  items: first the n_pairs pairs of a direction and its exact
// negation, then the n_single other directions; null: all M directions.
hipError_t launch_mm_far(qax_problem* p, const double* mu, int nrhs, const double* xhat, int64_t M, const int2* items,
                         int64_t n_pairs, int64_t n_single, int slots, double* partial) {
  MmTargets P = {xhat, 3, 1, M, items, n_pairs, p->d_pinfo, p->n_problems, 0};
  auto grid = [&](int64_t n, int per) {
    return dim3((unsigned)((n + per - 1) / per), (unsigned)slots, (unsigned)p->n_problems);
  };
  hipError_t e = hipSuccess;
  if (items && n_pairs)
    e = launch_mm_forms<MM_FAR, true>(p, nullptr, P, grid(n_pairs, MM_T / 2), mu, nrhs, partial);
  P.items = items ? items + n_pairs : nullptr;
  P.n_items = items ? n_single : M;
  if (e == hipSuccess && P.n_items)
    e = launch_mm_forms<MM_FAR, false>(p, nullptr, P, grid(P.n_items, MM_T), mu, nrhs, partial);
  return e;
}

}  // namespace qax
