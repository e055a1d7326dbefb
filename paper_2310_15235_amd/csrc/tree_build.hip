// Radiation tree construction on gfx950 (Section 2.3 and 2.6 of Wadsley,
// Baumschlager & Shen 2023): root cube, 63-bit Morton keys (21 bits per
// axis, x first), stable LSD radix sort, a radix tree whose nodes split at
// the first differing key bit (half-way along the longest axis of a cube or
// 2:1 box) down to buckets of at most leaf_size elements, node moments
// (luminosities, luminosity centre, bucket absorption) and per-direction
// transmission-averaged absorption.
//
// The topology comes from the sorted keys alone (Karras 2012, "Maximizing
// parallelism in the construction of BVHs, octrees, and k-d trees"): every
// internal node of the binary radix tree finds its range and split by itself,
// the ones too large for a bucket are kept, and a prefix sum over the first
// slots of the nodes numbers them in depth-first preorder, so a subtree is a
// contiguous index range.  Moments and transmission tables are reduced
// bottom-up, a workgroup per subtree of at most kSubtree elements and level by
// level above, with FP64 sums formed in a fixed order (buckets sum their
// elements in key order; a parent adds its two children), which makes every
// node moment independent of the launch shape.
//
// What bounds the build is the number of dependent steps, not bytes (4 MB at
// 2^18 elements of one band): before, one launch per level and step (200
// launches, the host reading the levels back every six), now some 30 with one
// readback.  Kernels of a build, before -> now: 4096 elements of one band 540 ->
// 137 us, 2^18 of three bands 1360 -> 355 us, 2^21 of two bands and 24 direction
// classes 3500 -> 1480 us.

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>

#include "trevr_internal.hpp"

namespace trevr {

// --------------------------------------------------------------- helpers
__device__ inline uint32_t f2ord(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float ord2f(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}
__device__ inline bool finite_pos(float v) { return isfinite(v) && v > 0.0f; }

// ------------------------------------------------------------- root cube
// Direction of a point of the octahedral map (not normalised).
__device__ inline void octahedral(float u, float v, float d[3]) {
  d[2] = 1.0f - fabsf(u) - fabsf(v);
  d[0] = u;
  d[1] = v;
  if (d[2] < 0.0f) {
    d[0] = copysignf(1.0f - fabsf(v), u);
    d[1] = copysignf(1.0f - fabsf(u), v);
  }
  const float inv = rsqrtf(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
  d[0] *= inv;
  d[1] *= inv;
  d[2] *= inv;
}

// Workgroup 0 zeroes the build's counters and, with a box from the caller,
// writes the header.  The others fill the table of candidate rays, one
// wavefront per (bin, group of 64 rays): the bin's angular radius is the
// farthest of 8 x 8 points of it from its middle, plus what lies between them
// (half a step's diagonal, 0.0063 of the map, which stretches angles up to
// threefold), and each step of the sine takes the rays within that angle and
// its own.
constexpr float kCandSlack = 0.02f;
static_assert(kCandSide == 32, "kCandSlack holds for bins of 1/16 of the map's half width");
__global__ void __launch_bounds__(256) k_init(TreeBufs tb, double bx, double by, double bz,
                                              double bL, int nray) {
  const int t = threadIdx.x;
  if (blockIdx.x == 0) {
    if (t < 3) { tb.bbox_u[t] = 0xFFFFFFFFu; tb.bbox_u[3 + t] = 0u; }
    if (t < 4) tb.err[t] = 0u;
    if (t < CNT_N) tb.counters[t] = 0ull;
    if (t < (int)(sizeof(BuildWords) / 4)) reinterpret_cast<uint32_t*>(tb.words)[t] = 0u;
    if (t == 0) tb.tsum[0] = 0u;
    if (t == 0 && bL > 0.0) {
      tb.hdr[0] = bx; tb.hdr[1] = by; tb.hdr[2] = bz; tb.hdr[3] = bL;
      tb.hdr[4] = ldexp(1.0, kKeyBits) / bL;
    }
    return;
  }
  const int lane = t & 63, groups = (nray + 63) / 64;
  const int w = (int)(blockIdx.x - 1) * 4 + (t >> 6);
  const int bin = w / groups, g = w % groups;
  if (bin >= kCandSide * kCandSide) return;
  constexpr float kWidth = 2.0f / kCandSide;
  const float u0 = -1.0f + kWidth * (float)(bin % kCandSide);
  const float v0 = -1.0f + kWidth * (float)(bin / kCandSide);
  float mid[3], d[3];
  octahedral(u0 + 0.5f * kWidth, v0 + 0.5f * kWidth, mid);
  octahedral(u0 + kWidth * (float)(lane & 7) / 7.0f, v0 + kWidth * (float)(lane >> 3) / 7.0f, d);
  float rad = acosf(fminf(1.0f, mid[0] * d[0] + mid[1] * d[1] + mid[2] * d[2]));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) rad = fmaxf(rad, __shfl_xor(rad, o));
  const int k = 64 * g + lane;
  float ang = 4.0f;   // past every limit: no such ray
  if (k < nray) {
    const double* n = tb.ray_n + 3 * k;
    const float dp = mid[0] * (float)n[0] + mid[1] * (float)n[1] + mid[2] * (float)n[2];
    ang = acosf(fmaxf(-1.0f, fminf(1.0f, dp)));
  }
  uint64_t mine = 0ull;
#pragma unroll
  for (int q = 0; q < kCandSin; ++q) {
    const uint64_t m = ballot64(ang <= rad + asinf((float)(q + 1) / kCandSin) + kCandSlack);
    if (lane == q) mine = m;
  }
  if (lane < kCandSin)
    tb.rcand[((size_t)lane * (kCandSide * kCandSide) + bin) * groups + g] = mine;
}

__global__ void __launch_bounds__(256) k_bbox(const float* x, const float* y, const float* z,
                                              int64_t n, uint32_t* bbox_u) {
  uint32_t mn[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, mx[3] = {0u, 0u, 0u};
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t v[3] = {f2ord(x[i]), f2ord(y[i]), f2ord(z[i])};
#pragma unroll
    for (int a = 0; a < 3; ++a) { mn[a] = min(mn[a], v[a]); mx[a] = max(mx[a], v[a]); }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    for (int o = 32; o > 0; o >>= 1) {
      mn[a] = min(mn[a], (uint32_t)__shfl_xor((int)mn[a], o));
      mx[a] = max(mx[a], (uint32_t)__shfl_xor((int)mx[a], o));
    }
  }
  // per workgroup, then one set of atomics (the six words share a cache line,
  // so atomics on them queue behind one another)
  __shared__ uint32_t part[4][6];
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      part[threadIdx.x >> 6][a] = mn[a];
      part[threadIdx.x >> 6][3 + a] = mx[a];
    }
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    const int a = threadIdx.x;
    uint32_t v = part[0][a];
    for (int w = 1; w < (int)(blockDim.x / 64); ++w)
      v = a < 3 ? min(v, part[w][a]) : max(v, part[w][a]);
    if (a < 3) atomicMin(&bbox_u[a], v);
    else atomicMax(&bbox_u[a], v);
  }
}

// hdr = {lo_x, lo_y, lo_z, L, 2^21 / L} without a box from the caller: L is
// the largest extent of the bounding box (1 if all elements coincide).
__global__ void k_header(const uint32_t* bbox_u, double* hdr) {
  if (threadIdx.x != 0) return;
  double lo[3], L = 0.0;
  for (int a = 0; a < 3; ++a) {
    lo[a] = (double)ord2f(bbox_u[a]);
    const double hi = (double)ord2f(bbox_u[3 + a]);
    L = fmax(L, hi - lo[a]);
  }
  if (L == 0.0) L = 1.0;
  hdr[0] = lo[0]; hdr[1] = lo[1]; hdr[2] = lo[2]; hdr[3] = L;
  hdr[4] = ldexp(1.0, kKeyBits) / L;
}

// ----------------------------------------------------------- Morton keys
// Bit b of a 21-bit word to bit 3b, and back.
__device__ inline uint64_t spread3(uint32_t v) {
  uint64_t x = v & 0x1FFFFFu;
  x = (x | (x << 32)) & 0x001F00000000FFFFull;
  x = (x | (x << 16)) & 0x001F0000FF0000FFull;
  x = (x | (x << 8)) & 0x100F00F00F00F00Full;
  x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
  x = (x | (x << 2)) & 0x1249249249249249ull;
  return x;
}
__device__ inline uint32_t compact3(uint64_t k, int a) {
  // bits of axis a sit at positions 3b + (2 - a)
  uint64_t x = (k >> (2 - a)) & 0x1249249249249249ull;
  x = (x | (x >> 2)) & 0x10C30C30C30C30C3ull;
  x = (x | (x >> 4)) & 0x100F00F00F00F00Full;
  x = (x | (x >> 8)) & 0x001F0000FF0000FFull;
  x = (x | (x >> 16)) & 0x001F00000000FFFFull;
  x = (x | (x >> 32)) & 0x1FFFFFull;
  return (uint32_t)x;
}

__device__ inline uint64_t morton_key(const double* hdr, float x, float y, float z) {
  const float X[3] = {x, y, z};
  const double scale = hdr[4];
  uint64_t k = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double u = floor(((double)X[a] - hdr[a]) * scale);
    if (!(u >= 0.0)) u = 0.0;
    if (u > 2097151.0) u = 2097151.0;
    k |= spread3((uint32_t)u) << (2 - a);
  }
  return k;
}

// Keys, the check of the inputs, the bits in which keys differ (for the
// sort) and each element packed into one record of rec_floats(B) floats
// {x, y, z, m, rho, (kappa, lum) per band}: the gather after the sort then
// touches one or two cache lines per element instead of one per array
// (2^21 elements, two bands: gather 338 -> 98 us, the keys 30 -> 57 with the
// records' 100 MB).
__global__ void __launch_bounds__(256) k_keys(const float* x, const float* y, const float* z,
                                              const float* m, const float* rho,
                                              const float* kappa, const float* lum, int64_t n,
                                              int B, TreeBufs tb) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  uint64_t diff = 0ull;
  if (i < n) {
    const float X[3] = {x[i], y[i], z[i]};
    const float mi = m[i], ri = rho[i];
    float4* rec = reinterpret_cast<float4*>(tb.rec + i * rec_floats(B));
    float4 q = make_float4(ri, 0.0f, 0.0f, 0.0f);
    rec[0] = make_float4(X[0], X[1], X[2], mi);
    bool ok = isfinite(X[0]) && isfinite(X[1]) && isfinite(X[2]) && finite_pos(mi) &&
              finite_pos(ri);
    int fill = 1, at = 1;
    for (int b = 0; b < B; ++b) {
      const float kv = kappa[(int64_t)b * n + i], lv = lum[(int64_t)b * n + i];
      ok = ok && isfinite(kv) && kv >= 0.0f && isfinite(lv) && lv >= 0.0f;
      if (fill == 1) {
        q.y = kv;
        q.z = lv;
        fill = 3;
      } else {
        q.w = kv;
        rec[at++] = q;
        q.x = lv;
        fill = 1;
      }
    }
    rec[at] = q;
    if (!ok) atomicOr(tb.err, ERR_DATA);
    const uint64_t k = morton_key(tb.hdr, X[0], X[1], X[2]);
    tb.keys_alt[i] = k;
    tb.starts[i] = 0u;
    if (i == n - 1) tb.starts[n] = 0u;
    diff = k ^ morton_key(tb.hdr, x[0], y[0], z[0]);
  }
  __shared__ unsigned long long part[4];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) diff |= (uint64_t)__shfl_xor((long long)diff, o);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = diff;
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned long long d = part[0] | part[1] | part[2] | part[3];
    // the atomic only for bits not seen set yet (a stale read shows fewer)
    if (d & ~__atomic_load_n(&tb.words->diff, __ATOMIC_RELAXED)) atomicOr(&tb.words->diff, d);
  }
}

// ------------------------------------------------------------- the sort
// Up to kSmallSort elements: one workgroup sorts in LDS, 8 bits a pass, the
// passes whose bits all keys share left out.  Each wavefront ranks its 256
// consecutive keys by matching digits (ballots), the counts per (wavefront,
// digit) are scanned, the keys move to the other buffer.  At 4096 elements
// the passes over global memory took 225 us in 24 launches of one or two
// workgroups, this one 36 us.
constexpr int kSmallSort = 4096;
__global__ void __launch_bounds__(1024) k_sort_small(int64_t n64, TreeBufs tb) {
  __shared__ uint64_t K[2][kSmallSort];
  __shared__ uint16_t V[2][kSmallSort];
  __shared__ uint32_t cnt[16][256];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, n = (int)n64;
  for (int i = t; i < n; i += 1024) {
    K[0][i] = tb.keys_alt[i];
    V[0][i] = (uint16_t)i;
  }
  const uint64_t diff = tb.words->diff;
  int cur = 0;
  for (int shift = 0; shift < 64; shift += 8) {
    if (((diff >> shift) & 255ull) == 0ull) continue;
    __syncthreads();
    for (int i = t; i < 16 * 256; i += 1024) (&cnt[0][0])[i] = 0u;
    __syncthreads();
    uint64_t k[4];
    uint32_t rk[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = w * 256 + r * 64 + lane;
      const bool valid = i < n;
      k[r] = valid ? K[cur][i] : 0ull;
      const uint32_t d = (uint32_t)(k[r] >> shift) & 255u;
      uint64_t mm = ballot64(valid);
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        const bool on = (d >> bit) & 1u;
        const uint64_t bb = ballot64(on);
        mm &= on ? bb : ~bb;
      }
      const uint32_t pre = cnt[w][d];
      wave_lds_sync();
      const int rank = mbcnt(mm);
      if (valid && rank == 0) cnt[w][d] = pre + (uint32_t)__popcll(mm);
      wave_lds_sync();
      rk[r] = pre + (uint32_t)rank;
    }
    __syncthreads();
    uint32_t run = 0;
    if (t < 256)
      for (int ww = 0; ww < 16; ++ww) run += cnt[ww][t];
    const uint32_t base = block_excl_u32(run, nullptr);
    if (t < 256) {
      run = base;
      for (int ww = 0; ww < 16; ++ww) {
        const uint32_t c = cnt[ww][t];
        cnt[ww][t] = run;
        run += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = w * 256 + r * 64 + lane;
      if (i < n) {
        const uint32_t p = cnt[w][(uint32_t)(k[r] >> shift) & 255u] + rk[r];
        K[cur ^ 1][p] = k[r];
        V[cur ^ 1][p] = V[cur][i];
      }
    }
    cur ^= 1;
  }
  __syncthreads();
  for (int i = t; i < n; i += 1024) {
    tb.keys[i] = K[cur][i];
    tb.vals[i] = V[cur][i];
  }
}

// More elements: stable LSD radix sort, 8 bits a pass, of the 32 highest
// bits in which keys differ (four passes over 4-byte keys); k_sort_finish
// then orders the few elements whose 32 bits agree.  When some run of those
// is long (elements crowded into 2^-10 of the varying extent) every later
// kernel of the build exits and the host builds again with all 64 bits
// sorted (WIDE: eight passes over 8-byte keys).
__device__ inline uint32_t top_bits(uint64_t k, uint64_t diff) {
  const int len = 64 - __clzll((long long)diff);   // varying bits
  return (uint32_t)(len > 32 ? k >> (len - 32) : k);
}
template <bool WIDE> struct SortKey { using type = uint32_t; };
template <> struct SortKey<true> { using type = uint64_t; };

// The key of pass `pass`: the first pass of the short sort reads the full
// keys in input order.
template <bool WIDE>
__device__ inline typename SortKey<WIDE>::type sort_key(const void* in, int64_t i, int pass,
                                                        uint64_t diff) {
  if (WIDE) return (typename SortKey<WIDE>::type)((const uint64_t*)in)[i];
  if (pass == 0) return (typename SortKey<WIDE>::type)top_bits(((const uint64_t*)in)[i], diff);
  return (typename SortKey<WIDE>::type)((const uint32_t*)in)[i];
}

template <bool WIDE, int ITEMS>
__global__ void __launch_bounds__(256) k_sort_hist(const void* in, int64_t n, int pass,
                                                   TreeBufs tb, int nblk) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0u;
  const uint64_t diff = tb.words->diff;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * (256 * ITEMS);
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t i = base + r * 256 + threadIdx.x;
    if (i < n)
      atomicAdd(&h[(uint32_t)(sort_key<WIDE>(in, i, pass, diff) >> (8 * pass)) & 255u], 1u);
  }
  __syncthreads();
  tb.hist[(int64_t)threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}

// Exclusive scan of one digit's counts over the tiles (one workgroup per
// digit) and the digit's total.
__global__ void __launch_bounds__(256) k_sort_rows(uint32_t* hist, uint32_t* dtot, int nblk) {
  __shared__ uint32_t wsum[4];
  uint32_t* a = hist + (int64_t)blockIdx.x * nblk;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  uint32_t carry = 0;
  for (int b0 = 0; b0 < nblk; b0 += 256) {
    const uint32_t v = b0 + t < nblk ? a[b0 + t] : 0u;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t u = (uint32_t)__shfl_up((int)incl, o);
      if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t pre = carry, tot = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q < w) pre += wsum[q];
      tot += wsum[q];
    }
    if (b0 + t < nblk) a[b0 + t] = pre + incl - v;
    carry += tot;
    __syncthreads();
  }
  if (t == 0) dtot[blockIdx.x] = carry;
}

template <bool WIDE, int ITEMS>
__global__ void __launch_bounds__(256) k_sort_scatter(const void* in, const uint32_t* vin,
                                                      void* out, uint32_t* vout, int64_t n,
                                                      int pass, TreeBufs tb, int nblk) {
  using Key = typename SortKey<WIDE>::type;
  __shared__ uint32_t run[256];
  __shared__ uint32_t wcnt[4][256];
  __shared__ uint32_t wsum[4];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const uint64_t diff = tb.words->diff;
  const int64_t base = (int64_t)blockIdx.x * (256 * ITEMS);
  Key k[ITEMS];
  uint32_t v[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t i = base + r * 256 + t;
    k[r] = i < n ? sort_key<WIDE>(in, i, pass, diff) : (Key)0;
    v[r] = i < n ? (pass == 0 ? (uint32_t)i : vin[i]) : 0u;
  }
  // first slot of digit t in this tile: the smaller digits, then the tiles
  // before this one
  {
    const uint32_t d = tb.dtot[t];
    uint32_t incl = d;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t u = (uint32_t)__shfl_up((int)incl, o);
      if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t pre = incl - d;
    for (int q = 0; q < w; ++q) pre += wsum[q];
    run[t] = pre + tb.hist[(int64_t)t * nblk + blockIdx.x];
    wcnt[0][t] = wcnt[1][t] = wcnt[2][t] = wcnt[3][t] = 0u;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const bool valid = base + r * 256 + t < n;
    const uint32_t d = (uint32_t)(k[r] >> (8 * pass)) & 255u;
    uint64_t mm = ballot64(valid);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const bool on = (d >> bit) & 1u;
      const uint64_t bb = ballot64(on);
      mm &= on ? bb : ~bb;
    }
    const int rank_w = mbcnt(mm);
    if (valid && rank_w == 0) wcnt[w][d] = (uint32_t)__popcll(mm);
    __syncthreads();
    if (valid) {
      uint32_t dst = run[d] + (uint32_t)rank_w;
      for (int ww = 0; ww < w; ++ww) dst += wcnt[ww][d];
      ((Key*)out)[dst] = k[r];
      vout[dst] = v[r];
    }
    __syncthreads();
    run[t] += wcnt[0][t] + wcnt[1][t] + wcnt[2][t] + wcnt[3][t];
    wcnt[0][t] = wcnt[1][t] = wcnt[2][t] = wcnt[3][t] = 0u;
    __syncthreads();
  }
}

// Full keys in sorted order.  After the short sort the first thread of a run
// of equal 32 bits orders the run by the full keys (stable: equal keys stay
// in input order); a run longer than kRunMax raises words->resort.  Uniform
// elements have runs of two at most (2^21 of them in 2^32 cells: 500 runs).
constexpr int kRunMax = 24;
__global__ void __launch_bounds__(256) k_sort_finish(int64_t n, TreeBufs tb, int wide) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (wide) {   // sorted in place: the full keys lie in keys_alt
    tb.keys[i] = tb.keys_alt[i];
    return;
  }
  const uint32_t* top = tb.top;
  const uint32_t k = top[i];
  const bool whole = (tb.words->diff >> 32) == 0ull;   // 32 bits are all that vary
  if (whole || ((i == 0 || top[i - 1] != k) && (i + 1 >= n || top[i + 1] != k))) {
    tb.keys[i] = tb.keys_alt[tb.vals[i]];
    return;
  }
  if (i > 0 && top[i - 1] == k) return;   // the run's first thread orders it
  int len = 1;
  while (len <= kRunMax && i + len < n && top[i + len] == k) ++len;
  if (len > kRunMax) {
    __atomic_store_n(&tb.words->resort, 1u, __ATOMIC_RELAXED);
    return;
  }
  for (int a = 0; a < len; ++a) {   // insertion sort in place
    const uint32_t v = tb.vals[i + a];
    const uint64_t kv = tb.keys_alt[v];
    int q = a;
    for (; q > 0 && tb.keys[i + q - 1] > kv; --q) {
      tb.keys[i + q] = tb.keys[i + q - 1];
      tb.vals[i + q] = tb.vals[i + q - 1];
    }
    tb.keys[i + q] = kv;
    tb.vals[i + q] = v;
  }
}

// ------------------------------------------------- sorted element arrays
__global__ void __launch_bounds__(256) k_gather(int64_t n, int B, TreeBufs tb) {
  const int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (s >= n || tb.words->resort) return;
  const uint32_t i = tb.vals[s];
  const float4* rec = reinterpret_cast<const float4*>(tb.rec + (int64_t)i * rec_floats(B));
  const float4 p = rec[0];
  float4 q = rec[1];
  tb.perm[s] = i;
  tb.x[s] = p.x;
  tb.y[s] = p.y;
  tb.z[s] = p.z;
  tb.m[s] = p.w;
  tb.rho[s] = q.x;
  tb.h[s] = cbrt((double)p.w / (double)q.x);   // element size, Section 2.1
  double lb = 0.0;
  for (int b = 0, at = 2; b < B; ++b) {
    float kv, lv;
    if ((b & 1) == 0) {
      kv = q.y;
      lv = q.z;
    } else {
      kv = q.w;
      q = rec[at++];
      lv = q.x;
    }
    tb.kappa[(int64_t)b * n + s] = kv;
    tb.lum[(int64_t)b * n + s] = lv;
    lb += (double)lv;
  }
  tb.lbol[s] = lb;
}

// ------------------------------------------------------------- topology
// A node of the radix tree is kept as a cell if it holds more than leaf_size
// elements and its keys are not all equal; the other children of kept nodes
// are the buckets.
__device__ inline bool kept_range(const uint64_t* keys, uint32_t f, uint32_t l, int leaf_size) {
  return l - f + 1u > (uint32_t)leaf_size && keys[f] != keys[l];
}

// Length of the common prefix of the keys of slots i and j, slots told apart
// by their index where keys are equal; -1 outside the array.
__device__ inline int common_prefix(const uint64_t* keys, int64_t n, uint64_t ki, int64_t i,
                                    int64_t j) {
  if (j < 0 || j >= n) return -1;
  const uint64_t x = ki ^ keys[j];
  if (x) return __clzll((long long)x);
  return 64 + __clz((int)((uint32_t)i ^ (uint32_t)j));
}

// Internal node i of the radix tree covers slots from i to r_end[i], split
// after slot r_split[i]; its internal children are the nodes r_split[i] and
// r_split[i] + 1, whose r_par gets i.  Nodes not kept get r_end = kNoNode.
// starts[f] counts the cells and buckets whose first slot is f.
constexpr uint32_t kNoNode = 0xFFFFFFFFu;
__global__ void __launch_bounds__(256) k_radix(int64_t n, int leaf_size, TreeBufs tb) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n || tb.words->resort) return;
  const uint64_t* keys = tb.keys;
  const uint64_t ki = keys[i];
  const int dn = common_prefix(keys, n, ki, i, i + 1), dp = common_prefix(keys, n, ki, i, i - 1);
  const int64_t d = dn > dp ? 1 : -1;
  const int dmin = dn > dp ? dp : dn;
  tb.r_end[i] = kNoNode;
  // more than leaf_size elements, or not a cell (the root's bounds are known)
  if (i == n - 1 || common_prefix(keys, n, ki, i, i + d * leaf_size) <= dmin) {
    if (i == 0) atomicAdd(&tb.starts[0], 1u);   // the whole tree is one bucket
    return;
  }
  int64_t lmax = 2 * (int64_t)leaf_size;
  while (common_prefix(keys, n, ki, i, i + lmax * d) > dmin) lmax *= 2;
  int64_t len = 0;
  for (int64_t s = lmax / 2; s >= 1; s /= 2)
    if (common_prefix(keys, n, ki, i, i + (len + s) * d) > dmin) len += s;
  // lmax need not be a power of two: close the last gap
  while (common_prefix(keys, n, ki, i, i + (len + 1) * d) > dmin) ++len;
  const int64_t j = i + len * d;
  const uint32_t f = (uint32_t)(d > 0 ? i : j), l = (uint32_t)(d > 0 ? j : i);
  const uint64_t k0 = keys[f], k1 = keys[l];
  if (k0 == k1) {   // equal keys: a bucket however many
    if (i == 0) atomicAdd(&tb.starts[0], 1u);
    return;
  }
  const uint64_t bit = 1ull << (63 - __clzll((long long)(k0 ^ k1)));
  uint32_t lo = f, hi = l;   // key[lo] lacks the bit, key[hi] has it
  while (hi - lo > 1u) {
    const uint32_t mid = lo + (hi - lo) / 2u;
    if (keys[mid] & bit) hi = mid; else lo = mid;
  }
  tb.r_end[i] = (uint32_t)j;
  tb.r_split[i] = lo;
  if (lo > f) tb.r_par[lo] = (uint32_t)i;
  if (hi < l) tb.r_par[hi] = (uint32_t)i;
  atomicAdd(&tb.starts[f], 1u);
  if (!kept_range(keys, f, lo, leaf_size)) atomicAdd(&tb.starts[f], 1u);
  if (!kept_range(keys, hi, l, leaf_size)) atomicAdd(&tb.starts[hi], 1u);
}

// Exclusive scan of `total` words in tiles of 16384, one workgroup each: in
// place within the tile, the tiles' sums to tsum.
constexpr int kScanTile = 1024 * kScanPer;
__global__ void __launch_bounds__(1024) k_scan_tiles(uint32_t* a, int64_t total, uint32_t* tsum) {
  const int64_t b = blockIdx.x * (int64_t)kScanTile;
  const int64_t m = total - b < kScanTile ? total - b : (int64_t)kScanTile;
  block_scan_u32(a + b, m, gridDim.x > 1 ? tsum + blockIdx.x : nullptr);
}

// Cells and buckets starting before slot f.
__device__ inline uint32_t starts_before(const TreeBufs& tb, uint32_t f) {
  return tb.starts[f] + tb.tsum[f / (uint32_t)kScanTile];
}

__device__ inline void put_node(const TreeBufs& tb, uint32_t p, uint64_t key, int lown, bool leaf,
                                uint2 link, uint32_t next, int depth, bool big) {
  uint32_t kk[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) kk[a] = compact3(key, a) >> (kKeyBits - nbits_axis(lown, a));
  tb.nk[p] = make_uint4(kk[0], kk[1], kk[2], (uint32_t)lown | (leaf ? META_LEAF : 0u));
  tb.nlink[p] = link;
  tb.next[p] = next;
  tb.depth[p] = (uint8_t)(depth | (big ? kDeepBig : 0));
}

// The kept nodes and their buckets in preorder.  A node comes after every
// node that starts before it and after its ancestors that start with it:
// its index is the prefix sum at its first slot plus the number of the
// latter, counted (with its depth) by climbing to the root.  Nodes of up to
// kSubtree elements below a larger one are listed as subtree roots.
//
// A workgroup strides over the slots and adds its counts per depth and its
// list of roots once: with a workgroup per 256 slots, their atomics on a few
// shared lines took most of 495 us at 2^21 elements (now 150).
__global__ void __launch_bounds__(256) k_nodes(int64_t n, int leaf_size, TreeBufs tb) {
  constexpr uint32_t kList = 1024, kMostNew = 3 * 256;
  __shared__ uint32_t lcnt[kMaxLevels + 3], lbig, nlist, lbase, list[kList];
  if (tb.words->resort) return;
  const int t = threadIdx.x;
  for (int k = t; k < kMaxLevels + 3; k += 256) lcnt[k] = 0u;
  if (t == 0) {
    lbig = 0u;
    nlist = 0u;
  }
  __syncthreads();
  const uint64_t* keys = tb.keys;
  auto flush = [&]() {   // the roots listed so far to the global list
    __syncthreads();
    if (t == 0 && nlist) lbase = atomicAdd(&tb.words->nroots, nlist);
    __syncthreads();
    for (uint32_t k = t; k < nlist; k += 256) tb.roots[lbase + k] = list[k];
    __syncthreads();
    if (t == 0) nlist = 0u;
    __syncthreads();
  };
  for (int64_t i0 = blockIdx.x * (int64_t)256; i0 < n; i0 += (int64_t)gridDim.x * 256) {
    const int64_t i = i0 + t;
    const uint32_t e = i < n ? tb.r_end[i] : kNoNode;
    if (i == 0 && e == kNoNode) {   // one bucket
      put_node(tb, 0u, keys[0], 0, true, make_uint2(0u, (uint32_t)n), 1u, 0, false);
      atomicAdd(&lcnt[0], 1u);
      list[atomicAdd(&nlist, 1u)] = 0u;
    }
    if (e != kNoNode) {
      const uint32_t f = min((uint32_t)i, e), l = max((uint32_t)i, e), g = tb.r_split[i];
      int depth = 0, lown = 0;
      uint32_t same = 0, pcount = 0;
      for (uint32_t j = (uint32_t)i; j != 0u && depth < kMaxLevels; ++depth) {
        const uint32_t q = tb.r_par[j], qe = tb.r_end[q];
        if (depth == 0) {
          const uint32_t gs = tb.r_split[q];
          lown = __clzll((long long)(keys[gs] ^ keys[gs + 1]));   // parent's split bit + 1
          pcount = max(q, qe) - min(q, qe) + 1u;
        }
        same += min(q, qe) == f ? 1u : 0u;
        j = q;
      }
      const int s = __clzll((long long)(keys[g] ^ keys[g + 1])) - 1;   // split bit
      const uint32_t count = l - f + 1u;
      const bool big = count > (uint32_t)kSubtree;
      const uint32_t p = starts_before(tb, f) + same, c1 = starts_before(tb, g + 1u);
      put_node(tb, p, keys[f], lown, false, make_uint2(c1, (uint32_t)s),
               starts_before(tb, l + 1u), depth, big);
      atomicAdd(&lcnt[depth], 1u);
      if (big) atomicMax(&lbig, (uint32_t)depth + 1u);
      else if (i == 0 || pcount > (uint32_t)kSubtree) list[atomicAdd(&nlist, 1u)] = p;
      const uint32_t cf[2] = {f, g + 1u}, cl[2] = {g, l}, cp[2] = {p + 1u, c1};
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (kept_range(keys, cf[q], cl[q], leaf_size)) continue;
        put_node(tb, cp[q], keys[cf[q]], s + 1, true, make_uint2(cf[q], cl[q] - cf[q] + 1u),
                 cp[q] + 1u, depth + 1, false);
        atomicAdd(&lcnt[depth + 1], 1u);
        if (big) list[atomicAdd(&nlist, 1u)] = cp[q];
      }
    }
    __syncthreads();
    const bool full = nlist > kList - kMostNew;   // uniform: a barrier on either side
    __syncthreads();
    if (full) flush();
  }
  flush();
  for (int k = t; k < kMaxLevels + 3; k += 256)
    if (lcnt[k]) atomicAdd(&tb.words->lcnt[k], lcnt[k]);
  if (t == 0 && lbig > __atomic_load_n(&tb.words->bigdepth, __ATOMIC_RELAXED))
    atomicMax(&tb.words->bigdepth, lbig);
}

// The nodes grouped by depth: levels[d] the index range of depth d in b_pre,
// b_lown and b_split.  Workgroup 0 also writes the level table and the
// counts the host reads back, and completes the device's DevTree.
__global__ void __launch_bounds__(256) k_levels(int64_t n, TreeBufs tb) {
  __shared__ uint32_t lbeg[kMaxLevels + 4], lcnt[kMaxLevels + 3], lbase[kMaxLevels + 3];
  BuildWords& bw = *tb.words;
  if (bw.resort) {
    if (blockIdx.x == 0 && threadIdx.x == 0) tb.info[0] = 1u;
    return;
  }
  const int t = threadIdx.x;
  if (t < kMaxLevels + 3) lcnt[t] = bw.lcnt[t];
  __syncthreads();
  if (t == 0) {
    uint32_t run = 0, d = 0;
    for (int k = 0; k < kMaxLevels + 3; ++k) {
      const uint32_t c = lcnt[k];
      lbeg[k] = run;
      run += c;
      if (c) d = (uint32_t)k + 1u;
    }
    lbeg[kMaxLevels + 3] = run;
    if (blockIdx.x == 0) {
      tb.info[0] = 0u;
      tb.info[1] = run;
      tb.info[2] = d;
      tb.info[3] = bw.bigdepth;
      tb.dev->num_nodes = (int64_t)run;
      tb.dev->depth = (int32_t)d;
    }
  }
  __syncthreads();
  if (blockIdx.x == 0 && t < kMaxLevels + 3) tb.levels[t] = make_uint2(lbeg[t], lbeg[t + 1]);
  const uint32_t total = lbeg[kMaxLevels + 3];
  for (uint32_t p0 = blockIdx.x * 256u; p0 < total; p0 += gridDim.x * 256u) {
    __syncthreads();
    if (t < kMaxLevels + 3) lcnt[t] = 0u;
    __syncthreads();
    const uint32_t p = p0 + (uint32_t)t;
    int d = 0;
    uint32_t rank = 0;
    if (p < total) {
      d = (int)(tb.depth[p] & (kDeepBig - 1u));
      rank = atomicAdd(&lcnt[d], 1u);
    }
    __syncthreads();
    if (t < kMaxLevels + 3 && lcnt[t]) lbase[t] = lbeg[t] + atomicAdd(&bw.lcur[t], lcnt[t]);
    __syncthreads();
    if (p < total) {
      const uint32_t i = lbase[d] + rank;
      const uint4 nk = tb.nk[p];
      tb.b_pre[i] = p;
      tb.b_lown[i] = (int32_t)(nk.w & 63u);
      tb.b_split[i] = (nk.w & META_LEAF) ? -1 : (int32_t)tb.nlink[p].y;
    }
  }
}

// --------------------------------------------------------------- moments
// Luminosity centre sl/lbol, the box centre when dark, and the node's flags.
__device__ inline void node_done(const TreeBufs& tb, uint32_t p, const double sl[3], double lbol,
                                 double kmass) {
  uint4 nk = tb.nk[p];
  double lo[3], hi[3];
  node_box(tb.hdr, nk, lo, hi);
  double c[3];
  for (int a = 0; a < 3; ++a) c[a] = (lbol > 0.0) ? sl[a] / lbol : 0.5 * (lo[a] + hi[a]);
  tb.sl[p] = make_double4(sl[0], sl[1], sl[2], lbol);
  tb.kmass[p] = kmass;
  tb.cen[p] = make_double4(c[0], c[1], c[2], lbol);
  tb.nk[p].w = nk.w | (lbol > 0.0 ? META_LUM : 0u) | (kmass > 0.0 ? META_ABS : 0u);
}

// One of a bucket's B + 1 sums over its elements in key order.  Role b < B:
// the luminosity and the absorption sum(kappa m) / sum(m / rho) (Section 2.6)
// of band b, the same in every direction; role B: the luminosity centre and
// the absorbing mass.  Eight elements' values are loaded before they are
// added, so a role waits on memory a few times and not once per element.
__device__ inline void leaf_role(const TreeBufs& tb, uint32_t p, int role, int64_t n, int B,
                                 int nclass) {
  const uint2 lk = tb.nlink[p];
  const uint32_t end = lk.x + lk.y;
  constexpr int kLoad = 8;
  if (role < B) {
    const float* kap = tb.kappa + (int64_t)role * n;
    const float* lum = tb.lum + (int64_t)role * n;
    double Lb = 0.0, kmv = 0.0, vol = 0.0;
    for (uint32_t s0 = lk.x; s0 < end; s0 += kLoad) {
      float m[kLoad], r[kLoad], kv[kLoad], lv[kLoad];
#pragma unroll
      for (int k = 0; k < kLoad; ++k) {
        const uint32_t s = min(s0 + (uint32_t)k, end - 1u);
        m[k] = tb.m[s];
        r[k] = tb.rho[s];
        kv[k] = kap[s];
        lv[k] = lum[s];
      }
#pragma unroll
      for (int k = 0; k < kLoad; ++k) {
        if (s0 + (uint32_t)k >= end) break;
        const double ms = (double)m[k];
        Lb += (double)lv[k];
        kmv += (double)kv[k] * ms;
        vol += ms / (double)r[k];
      }
    }
    tb.Lb[(int64_t)p * B + role] = Lb;
    const double ab = kmv / vol;
    const int64_t row = (int64_t)p * nclass * B + role;
    for (int c = 0; c < nclass; ++c) {
      tb.alpha64[row + (int64_t)c * B] = ab;
      tb.alpha32[row + (int64_t)c * B] = (float)ab;
    }
    return;
  }
  double sl[3] = {0.0, 0.0, 0.0}, lbol = 0.0, kmass = 0.0;
  for (uint32_t s0 = lk.x; s0 < end; s0 += kLoad) {
    float x[kLoad], y[kLoad], z[kLoad];
    double lb[kLoad];
#pragma unroll
    for (int k = 0; k < kLoad; ++k) {
      const uint32_t s = min(s0 + (uint32_t)k, end - 1u);
      x[k] = tb.x[s];
      y[k] = tb.y[s];
      z[k] = tb.z[s];
      lb[k] = tb.lbol[s];
    }
#pragma unroll
    for (int k = 0; k < kLoad; ++k) {
      if (s0 + (uint32_t)k >= end) break;
      lbol += lb[k];
      sl[0] += lb[k] * (double)x[k];
      sl[1] += lb[k] * (double)y[k];
      sl[2] += lb[k] * (double)z[k];
    }
  }
  for (uint32_t s = lk.x; s < end; ++s) {
    const double ms = (double)tb.m[s];
    for (int b = 0; b < B; ++b) kmass += (double)tb.kappa[(int64_t)b * n + s] * ms;
  }
  node_done(tb, p, sl, lbol, kmass);
}

// One of a cell's nclass x B + 1 steps from its two children.  Role c B + b:
// the transmission average of band b in direction class c -- the children
// combine on the split box, then the result grows through the empty prefix
// boxes up to the owned box (empty space is vacuum); with `linear`
// (TREVR_ABSORPTION_AVG) the combine is the linear volume-weighted mean
// instead.  Role nclass x B: the moments.
__device__ inline void cell_role(const TreeBufs& tb, uint32_t p, int role, int B, int nclass,
                                 int linear) {
  const uint2 lk = tb.nlink[p];
  const uint32_t p0 = p + 1u, p1 = lk.x;
  if (role == nclass * B) {
    for (int b = 0; b < B; ++b)
      tb.Lb[(int64_t)p * B + b] = tb.Lb[(int64_t)p0 * B + b] + tb.Lb[(int64_t)p1 * B + b];
    const double4 s0 = tb.sl[p0], s1 = tb.sl[p1];
    const double sl[3] = {s0.x + s1.x, s0.y + s1.y, s0.z + s1.z};
    node_done(tb, p, sl, s0.w + s1.w, tb.kmass[p0] + tb.kmass[p1]);
    return;
  }
  const int s = (int)lk.y, l = (int)(tb.nk[p].w & 63u), c = role / B;
  const int64_t row = (int64_t)nclass * B;
  const double a1 = tb.alpha64[p0 * row + role], a2 = tb.alpha64[p1 * row + role];
  double A;
  if (linear) {
    A = combine_linear(a1, a2);
    for (int mm = s - 1; mm >= l; --mm) A = combine_linear(A, 0.0);
  } else {
    const double L = tb.hdr[3];
    A = combine64(&tb.geom[((int64_t)s * nclass + c) * 3], L, a1, a2);
    for (int mm = s - 1; mm >= l; --mm)
      A = combine64(&tb.geom[((int64_t)mm * nclass + c) * 3], L, A, 0.0);
  }
  tb.alpha64[p * row + role] = A;
  tb.alpha32[p * row + role] = (float)A;
}

// Subtrees of at most kSubtree elements, a workgroup each: its buckets, then
// its cells from the deepest level up, a barrier between levels (the
// children's values were stored by the same workgroup).  One launch for some
// ten levels; level by level over the whole tree, moments and averages took 528
// us in 50 launches (2^18 elements, three bands), now 91 here and 92 in k_cells.
__global__ void __launch_bounds__(256) k_subtrees(int64_t n, int B, int nclass, int linear,
                                                  TreeBufs tb) {
  constexpr int kMost = 2 * kSubtree;
  __shared__ uint16_t order[kMost];
  // bins: the buckets, then the cells by relative depth (at most 63 levels of
  // cells: a key has 63 bits to split at)
  __shared__ uint32_t cnt[64], cur[64];
  if (tb.words->resort) return;
  const int t = threadIdx.x;
  const uint32_t nroots = tb.words->nroots, roles = (uint32_t)(nclass * B + 1);
  for (uint32_t q = blockIdx.x; q < nroots; q += gridDim.x) {
    const uint32_t p0 = tb.roots[q], m = tb.next[p0] - p0;
    const int d0 = (int)(tb.depth[p0] & (kDeepBig - 1u));
    __syncthreads();
    if (t < 64) cnt[t] = 0u;
    __syncthreads();
    for (uint32_t k = t; k < m; k += 256) {
      const bool leaf = (tb.nk[p0 + k].w & META_LEAF) != 0u;
      atomicAdd(&cnt[leaf ? 0 : 1 + (int)(tb.depth[p0 + k] & (kDeepBig - 1u)) - d0], 1u);
    }
    __syncthreads();
    if (t < 64) {
      const uint32_t c = cnt[t];
      uint32_t incl = c;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = (uint32_t)__shfl_up((int)incl, o);
        if (t >= o) incl += u;
      }
      cnt[t] = cur[t] = incl - c;
    }
    __syncthreads();
    for (uint32_t k = t; k < m; k += 256) {
      const bool leaf = (tb.nk[p0 + k].w & META_LEAF) != 0u;
      order[atomicAdd(&cur[leaf ? 0 : 1 + (int)(tb.depth[p0 + k] & (kDeepBig - 1u)) - d0], 1u)] =
          (uint16_t)k;
    }
    __syncthreads();
    const uint32_t nleaf = cur[0];
    for (uint32_t w = t; w < nleaf * (uint32_t)(B + 1); w += 256)
      leaf_role(tb, p0 + order[w / (uint32_t)(B + 1)], (int)(w % (uint32_t)(B + 1)), n, B, nclass);
    int top = 63;
    while (top > 0 && cur[top] == cnt[top]) --top;
    for (int d = top; d >= 1; --d) {
      __syncthreads();
      const uint32_t b = cnt[d], work = (cur[d] - b) * roles;
      for (uint32_t w = t; w < work; w += 256)
        cell_role(tb, p0 + order[b + w / roles], (int)(w % roles), B, nclass, linear);
    }
  }
}

// The larger cells of levels dhi down to dlo, one thread per (cell, role):
// several levels in one launch of one workgroup (a barrier between them)
// where they are small, one level per launch otherwise.
__global__ void __launch_bounds__(1024) k_cells(int dhi, int dlo, int B, int nclass, int linear,
                                                TreeBufs tb) {
  for (int d = dhi; d >= dlo; --d) {
    const uint2 lv = tb.levels[d];
    const uint32_t roles = (uint32_t)(nclass * B + 1);
    const int64_t work = (int64_t)(lv.y - lv.x) * roles;
    for (int64_t w = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; w < work;
         w += (int64_t)gridDim.x * blockDim.x) {
      const uint32_t p = tb.b_pre[lv.x + (uint32_t)(w / roles)];
      if (tb.depth[p] & kDeepBig) cell_role(tb, p, (int)(w % roles), B, nclass, linear);
    }
    __syncthreads();
  }
}

// Complex source model (Section 2.7, eq. srccomb, Fig. sourcecombine): the
// nodes of one level, one thread per (node, direction k over all N_ray).
// The ray from the node's luminosity centre c along n_k runs to the edge of
// the node's box (length d).  A bucket's ray sees the bucket absorption.  A
// merged node brings its children's rays to the same projected stopping
// point, the plane through c + d n_k normal to n_k: child i needs length
// D_i = d + (c - c_i).n_k, of which its own ray covers up to d_i (clipped
// when shorter, nothing when D_i <= 0) and the rest crosses the node with
// its transmission-averaged absorption in direction k; the optical depths
// combine so that attenuated luminosities add, per band:
//   L e^{-tau} = L_1 e^{-tau_1} + L_2 e^{-tau_2},
// and the node keeps alpha = tau / d (zero when d = 0 or L = 0).  Runs after
// k_subtrees and k_cells, level by level (it reads the transmission averages).
__global__ void k_csrc(TreeBufs tb, uint32_t lb, uint32_t le, int B, int nclass, int nray) {
  const int64_t gid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (gid >= (int64_t)(le - lb) * nray) return;
  const uint32_t i = lb + (uint32_t)(gid / nray);
  const int k = (int)(gid % nray);
  const uint32_t p = tb.b_pre[i];
  const double4 cp = tb.cen[p];
  const double c[3] = {cp.x, cp.y, cp.z};
  double lo[3], hi[3];
  node_box(tb.hdr, tb.nk[p], lo, hi);
  const double* nv = &tb.ray_n[3 * k];
  double dn = INFINITY;
  for (int a = 0; a < 3; ++a) {
    if (nv[a] > 0.0) dn = fmin(dn, (hi[a] - c[a]) / nv[a]);
    else if (nv[a] < 0.0) dn = fmin(dn, (lo[a] - c[a]) / nv[a]);
  }
  dn = fmax(dn, 0.0);
  tb.csrc_d[(int64_t)p * nray + k] = dn;
  double* out = &tb.csrc_a[((int64_t)p * nray + k) * B];
  if (tb.b_split[i] < 0) {
    for (int b = 0; b < B; ++b) out[b] = tb.alpha64[(int64_t)p * nclass * B + b];
    return;
  }
  const uint32_t ch[2] = {p + 1u, tb.nlink[p].x};
  double Dq[2], dq[2];
  for (int q = 0; q < 2; ++q) {
    const double4 cc = tb.cen[ch[q]];
    double D = dn;
    D += (c[0] - cc.x) * nv[0];
    D += (c[1] - cc.y) * nv[1];
    D += (c[2] - cc.z) * nv[2];
    Dq[q] = D;
    dq[q] = tb.csrc_d[(int64_t)ch[q] * nray + k];
  }
  const int cls = tb.ray_class[k];
  for (int b = 0; b < B; ++b) {
    const double Ln = tb.Lb[(int64_t)p * B + b];
    double al = 0.0;
    if (Ln > 0.0 && dn > 0.0) {
      const double aext = tb.alpha64[((int64_t)p * nclass + cls) * B + b];
      double tau[2], w[2];
      for (int q = 0; q < 2; ++q) {
        w[q] = tb.Lb[(int64_t)ch[q] * B + b] / Ln;
        const double ai = tb.csrc_a[((int64_t)ch[q] * nray + k) * B + b];
        if (!(Dq[q] > 0.0)) tau[q] = 0.0;
        else if (Dq[q] <= dq[q]) tau[q] = ai * Dq[q];
        else tau[q] = ai * dq[q] + aext * (Dq[q] - dq[q]);
      }
      int first = -1;
      for (int q = 0; q < 2; ++q)
        if (w[q] > 0.0 && (first < 0 || tau[q] < tau[first])) first = q;
      double sum = 0.0;
      for (int q = 0; q < 2; ++q)
        if (w[q] > 0.0) sum += w[q] * exp(-(tau[q] - tau[first]));
      al = (tau[first] - log(sum)) / dn;
    }
    out[b] = al;
  }
}

// ======================================================== host side
static void healpix_centres(int N, std::vector<double>& v) {
  v.assign(3 * 12 * N * N, 0.0);
  int k = 0;
  for (int i = 1; i <= 4 * N - 1; ++i) {
    double z, dphi, phi0;
    int cnt;
    if (i < N) {
      z = 1.0 - (double)i * i / (3.0 * N * N);
      cnt = 4 * i;
      dphi = kPi / (2.0 * i);
      phi0 = 0.5 * dphi;
    } else if (i <= 3 * N) {
      z = 4.0 / 3.0 - 2.0 * i / (3.0 * N);
      cnt = 4 * N;
      dphi = kPi / (2.0 * N);
      phi0 = ((i - N) % 2 == 0) ? 0.5 * dphi : 0.0;
    } else {
      const int ii = 4 * N - i;
      z = -(1.0 - (double)ii * ii / (3.0 * N * N));
      cnt = 4 * ii;
      dphi = kPi / (2.0 * ii);
      phi0 = 0.5 * dphi;
    }
    const double st = std::sqrt((1.0 - z) * (1.0 + z));
    for (int j = 0; j < cnt; ++j, ++k) {
      const double phi = phi0 + j * dphi;
      v[3 * k] = st * std::cos(phi);
      v[3 * k + 1] = st * std::sin(phi);
      v[3 * k + 2] = z;
    }
  }
}

// Ray-volume weights and chord of a box of sides s split across axis a,
// for lines along n (Section 2.6): V12 is the volume of lines crossing the
// joining face, V1 = V2 = (V - V12)/2, d the chord through the centre.
static void combine_geometry(const double s[3], int a, const double n[3], double out[3]) {
  const double V = s[0] * s[1] * s[2];
  double V12 = 0.0;
  if (n[a] != 0.0) {
    const int b = (a + 1) % 3, c = (a + 2) % 3;
    const double tb = std::fabs(n[b] / n[a]), tc = std::fabs(n[c] / n[a]);
    double U = 0.5 * s[a];
    if (tb > 0.0) U = std::min(U, s[b] / tb);
    if (tc > 0.0) U = std::min(U, s[c] / tc);
    V12 = 2.0 * (s[b] * s[c] * U - (s[b] * tc + s[c] * tb) * U * U / 2.0 + tb * tc * U * U * U / 3.0);
  }
  const double w1 = std::max(0.0, (V - V12) / 2.0) / V;
  const double w12 = std::min(1.0, V12 / V);
  double d = INFINITY;
  for (int c = 0; c < 3; ++c)
    if (n[c] != 0.0) d = std::min(d, s[c] / std::fabs(n[c]));
  out[0] = (w1 > 0.0) ? std::log(w1) : -INFINITY;
  out[1] = (w12 > 0.0) ? std::log(w12) : -INFINITY;
  out[2] = d;
}

DirTables make_dir_tables(int nside) {
  DirTables t;
  t.nside = nside;
  t.nray = 12 * nside * nside;
  healpix_centres(nside, t.ray_n);
  t.ray_class.assign(t.nray, -1);
  std::vector<int> rep;
  for (int k = 0; k < t.nray; ++k) {
    const double* v = &t.ray_n[3 * k];
    int found = -1;
    for (size_t c = 0; c < rep.size() && found < 0; ++c) {
      const double* w = &t.ray_n[3 * rep[c]];
      if (std::fabs(std::fabs(v[0]) - std::fabs(w[0])) < 1e-12 &&
          std::fabs(std::fabs(v[1]) - std::fabs(w[1])) < 1e-12 &&
          std::fabs(std::fabs(v[2]) - std::fabs(w[2])) < 1e-12)
        found = (int)c;
    }
    if (found < 0) {
      found = (int)rep.size();
      rep.push_back(k);
    }
    t.ray_class[k] = found;
  }
  t.nclass = (int)rep.size();
  // antipodes: HEALPix centres come in opposite pairs, so -n_k is the centre
  // nearest to it
  t.ray_anti.assign(t.nray, 0);
  for (int k = 0; k < t.nray; ++k) {
    double best = INFINITY;
    for (int j = 0; j < t.nray; ++j) {
      double d2 = 0.0;
      for (int a = 0; a < 3; ++a) {
        const double u = t.ray_n[3 * j + a] + t.ray_n[3 * k + a];
        d2 += u * u;
      }
      if (d2 < best) { best = d2; t.ray_anti[k] = j; }
    }
  }
  t.geom.assign((size_t)kMaxLevels * t.nclass * 3, 0.0);
  for (int l = 0; l < kMaxLevels; ++l) {
    double s[3];
    for (int a = 0; a < 3; ++a) s[a] = std::ldexp(1.0, -nbits_axis(l, a));
    for (int c = 0; c < t.nclass; ++c)
      combine_geometry(s, l % 3, &t.ray_n[3 * rep[c]], &t.geom[((size_t)l * t.nclass + c) * 3]);
  }
  t.block.assign(dir_block(t.nray, t.nclass), 0.0);
  std::copy(t.ray_n.begin(), t.ray_n.end(), t.block.begin());
  std::copy(t.geom.begin(), t.geom.end(), t.block.begin() + t.ray_n.size());
  int32_t* ints = reinterpret_cast<int32_t*>(t.block.data() + t.ray_n.size() + t.geom.size());
  std::copy(t.ray_class.begin(), t.ray_class.end(), ints);
  std::copy(t.ray_anti.begin(), t.ray_anti.end(), ints + t.nray);
  return t;
}

namespace {
constexpr int kSides = 5;   // N_side 1, 2, 4, 8, 16
static_assert((1 << (kSides - 1)) == kMaxNside, "one set of tables per N_side");
std::mutex g_dir_mu;
std::unique_ptr<DirTables> g_dirs[kSides];
double* g_dir_pinned[kSides] = {};
std::mutex g_pin_mu;
std::vector<uint32_t*> g_pins;
constexpr size_t kPinsKept = 16;   // 2 KiB each
int side_index(int nside) {
  int k = 0;
  while ((1 << k) < nside && k < kSides - 1) ++k;
  return k;
}
}  // namespace

const DirTables& dir_tables(int nside) {
  std::lock_guard<std::mutex> g(g_dir_mu);
  std::unique_ptr<DirTables>& d = g_dirs[side_index(nside)];
  if (!d) d.reset(new DirTables(make_dir_tables(nside)));
  return *d;
}

const double* dir_block_pinned(int nside) {
  const DirTables& d = dir_tables(nside);
  std::lock_guard<std::mutex> g(g_dir_mu);
  double*& p = g_dir_pinned[side_index(nside)];
  if (!p) {
    void* q = nullptr;
    if (hipHostMalloc(&q, d.block.size() * sizeof(double), hipHostMallocPortable) != hipSuccess) {
      (void)hipGetLastError();
      return d.block.data();
    }
    p = (double*)q;
    std::copy(d.block.begin(), d.block.end(), p);
  }
  return p;
}

trevr_status pinned_take(uint32_t** out) {
  {
    std::lock_guard<std::mutex> g(g_pin_mu);
    if (!g_pins.empty()) {
      *out = g_pins.back();
      g_pins.pop_back();
      return TREVR_OK;
    }
  }
  return hip_check(hipHostMalloc((void**)out, kHostWords * sizeof(uint32_t), hipHostMallocPortable),
                   "hipHostMalloc");
}

void pinned_give(uint32_t* block) {
  {
    std::lock_guard<std::mutex> g(g_pin_mu);
    if (g_pins.size() < kPinsKept) {
      g_pins.push_back(block);
      return;
    }
  }
  (void)hipHostFree(block);
}

size_t layout_tree(const trevr_params& p, int64_t n, int nclass, void* base, TreeBufs* o) {
  Carve cv(base);
  TreeBufs t{};
  const int64_t M = 2 * n;
  const int B = p.n_bands;
  const int nray = 12 * p.nside * p.nside;
  t.hdr = cv.take<double>(8);
  t.bbox_u = cv.take<uint32_t>(8);
  t.err = cv.take<uint32_t>(4);
  t.counters = cv.take<unsigned long long>(CNT_N);
  t.words = cv.take<BuildWords>(1);
  t.keys = cv.take<uint64_t>(n);
  t.keys_alt = cv.take<uint64_t>(n);
  t.vals = cv.take<uint32_t>(n);
  t.vals_alt = cv.take<uint32_t>(n);
  t.top = cv.take<uint32_t>(n);
  t.top_alt = cv.take<uint32_t>(n);
  t.hist = cv.take<uint32_t>(256 * sort_tiles(n));
  t.dtot = cv.take<uint32_t>(256);
  t.rec = cv.take<float>((size_t)n * rec_floats(B));
  t.starts = cv.take<uint32_t>(n + 1);
  t.tsum = cv.take<uint32_t>(n / (1024 * kScanPer) + 2);
  t.roots = cv.take<uint32_t>(n);
  t.r_end = t.top;          // free once the elements are gathered
  t.r_split = t.top_alt;
  t.r_par = t.vals_alt;
  t.x = cv.take<float>(n);
  t.y = cv.take<float>(n);
  t.z = cv.take<float>(n);
  t.m = cv.take<float>(n);
  t.rho = cv.take<float>(n);
  t.kappa = cv.take<float>(B * n);
  t.lum = cv.take<float>(B * n);
  t.h = cv.take<double>(n);
  t.lbol = cv.take<double>(n);
  t.perm = cv.take<uint32_t>(n);
  t.b_pre = cv.take<uint32_t>(M);
  t.b_lown = cv.take<int32_t>(M);
  t.b_split = cv.take<int32_t>(M);
  t.nk = cv.take<uint4>(M);
  t.nlink = cv.take<uint2>(M);
  t.next = cv.take<uint32_t>(M);
  t.depth = cv.take<uint8_t>(M);
  t.cen = cv.take<double4>(M);
  t.sl = cv.take<double4>(M);
  t.Lb = cv.take<double>(M * B);
  t.kmass = cv.take<double>(M);
  t.alpha64 = cv.take<double>(M * nclass * B);
  t.alpha32 = cv.take<float>(M * nclass * B);
  // the direction tables, laid out as DirTables::block
  t.ray_n = cv.take<double>(dir_block(nray, nclass));
  t.geom = t.ray_n ? t.ray_n + 3 * nray : nullptr;
  t.ray_class = t.ray_n ? (int32_t*)(t.geom + (size_t)kMaxLevels * nclass * 3) : nullptr;
  t.ray_anti = t.ray_n ? t.ray_class + nray : nullptr;
  t.rcand = cv.take<uint64_t>((size_t)kCandSin * kCandSide * kCandSide * ((nray + 63) / 64));
  t.csrc_d = nullptr;
  t.csrc_a = nullptr;
  if (p.flags & TREVR_COMPLEX_SRC) {
    t.csrc_d = cv.take<double>(M * nray);
    t.csrc_a = cv.take<double>(M * nray * B);
  }
  t.dev = cv.take<DevTree>(1);
  t.levels = cv.take<uint2>(kMaxLevels + 3 + kInfoWords / 2);
  t.info = base ? reinterpret_cast<uint32_t*>(t.levels + kMaxLevels + 3) : nullptr;
  if (o) *o = t;
  return cv.off + 256;
}

static inline unsigned grid_for(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

#define TREVR_LAUNCH_CHECK(what)                                               \
  do {                                                                         \
    if ((rc = hip_check(hipGetLastError(), what)) != TREVR_OK) return rc;      \
  } while (0)

// The radix passes.  Tiles of 1024 elements up to kSortTileSwitch (at 2^18
// elements 256 tiles, one per CU; tiles of 4096 left three quarters of the
// chip idle), of 4096 above, where the counts per tile weigh more.
template <bool WIDE, int ITEMS>
static trevr_status sort_pass(trevr_tree* T, const void* in, const uint32_t* vin, void* out,
                              uint32_t* vout, int pass) {
  trevr_status rc;
  const TreeBufs& tb = T->buf;
  const int nblk = (int)((T->n + 256 * ITEMS - 1) / (256 * ITEMS));
  k_sort_hist<WIDE, ITEMS><<<nblk, 256, 0, T->stream>>>(in, T->n, pass, tb, nblk);
  TREVR_LAUNCH_CHECK("k_sort_hist");
  k_sort_rows<<<256, 256, 0, T->stream>>>(tb.hist, tb.dtot, nblk);
  TREVR_LAUNCH_CHECK("k_sort_rows");
  k_sort_scatter<WIDE, ITEMS><<<nblk, 256, 0, T->stream>>>(in, vin, out, vout, T->n, pass, tb,
                                                          nblk);
  TREVR_LAUNCH_CHECK("k_sort_scatter");
  return rc;
}

template <bool WIDE> static trevr_status sort_passes(trevr_tree* T) {
  const TreeBufs& tb = T->buf;
  const void* in = tb.keys_alt;   // full keys in input order
  const uint32_t* vin = nullptr;
  for (int pass = 0; pass < (WIDE ? 8 : 4); ++pass) {
    const bool odd = pass & 1;
    void* out = WIDE ? (void*)(odd ? tb.keys_alt : tb.keys) : (void*)(odd ? tb.top : tb.top_alt);
    uint32_t* vout = odd ? tb.vals : tb.vals_alt;
    const trevr_status rc = T->n <= kSortTileSwitch
                                ? sort_pass<WIDE, 4>(T, in, vin, out, vout, pass)
                                : sort_pass<WIDE, 16>(T, in, vin, out, vout, pass);
    if (rc != TREVR_OK) return rc;
    in = out;
    vin = vout;
  }
  return TREVR_OK;
}

trevr_status build_tree_impl(trevr_tree* T, const float* x, const float* y, const float* z,
                             const float* m, const float* rho, const float* kappa,
                             const float* lum) {
  const int64_t n = T->n;
  const int B = T->B;
  const int nclass = T->nclass;
  TreeBufs& tb = T->buf;
  hipStream_t st = T->stream;
  trevr_status rc;

  // the device's DevTree (k_levels completes it) and the direction tables,
  // both from pinned memory
  static_assert(sizeof(DevTree) <= kHostWords * sizeof(uint32_t) / 2, "fits the second half");
  uint32_t* up = T->host_u32 + kHostWords / 2;
  std::memcpy(up, &T->dev, sizeof(DevTree));
  if ((rc = hip_check(hipMemcpyAsync(tb.dev, up, sizeof(DevTree), hipMemcpyHostToDevice, st),
                      "copy tree table")) != TREVR_OK) return rc;
  if ((rc = hip_check(hipMemcpyAsync(tb.ray_n, dir_block_pinned(T->p.nside),
                                     sizeof(double) * T->dirs->block.size(),
                                     hipMemcpyHostToDevice, st), "copy direction tables")) !=
      TREVR_OK)
    return rc;

  const double* bx = T->p.box;
  const int cand_waves = kCandSide * kCandSide * ((T->nray + 63) / 64);
  k_init<<<1 + (cand_waves + 3) / 4, 256, 0, st>>>(tb, bx[0], bx[1], bx[2], bx[3], T->nray);
  TREVR_LAUNCH_CHECK("k_init");
  if (!(bx[3] > 0.0)) {
    k_bbox<<<std::min<int64_t>(64, grid_for(n, 256)), 256, 0, st>>>(x, y, z, n, tb.bbox_u);
    TREVR_LAUNCH_CHECK("k_bbox");
    k_header<<<1, 64, 0, st>>>(tb.bbox_u, tb.hdr);
    TREVR_LAUNCH_CHECK("k_header");
  }
  const unsigned gn = grid_for(n, 256);
  k_keys<<<gn, 256, 0, st>>>(x, y, z, m, rho, kappa, lum, n, B, tb);
  TREVR_LAUNCH_CHECK("k_keys");
  const int linear = (T->p.flags & TREVR_ABSORPTION_AVG) ? 1 : 0;
  uint32_t* info = T->host_u32 + 2 * (kMaxLevels + 3);
  for (bool wide = false;; wide = true) {
    // an even number of passes ends in the buffers it started from
    if (n <= kSmallSort) {
      k_sort_small<<<1, 1024, 0, st>>>(n, tb);
      TREVR_LAUNCH_CHECK("k_sort_small");
    } else {
      rc = wide ? sort_passes<true>(T) : sort_passes<false>(T);
      if (rc != TREVR_OK) return rc;
      k_sort_finish<<<gn, 256, 0, st>>>(n, tb, wide ? 1 : 0);
      TREVR_LAUNCH_CHECK("k_sort_finish");
    }
    k_gather<<<gn, 256, 0, st>>>(n, B, tb);
    TREVR_LAUNCH_CHECK("k_gather");

    // topology, then the moments of the small subtrees; the host reads the
    // counts back while those run
    k_radix<<<gn, 256, 0, st>>>(n, T->p.leaf_size, tb);
    TREVR_LAUNCH_CHECK("k_radix");
    const unsigned tiles = grid_for(n + 1, kScanTile);
    k_scan_tiles<<<tiles, 1024, 0, st>>>(tb.starts, n + 1, tb.tsum);
    TREVR_LAUNCH_CHECK("k_scan_tiles");
    if (tiles > 1) {   // (one tile: its offset is the zero of k_init)
      k_scan_u32<<<1, 1024, 0, st>>>(tb.tsum, tiles, nullptr);
      TREVR_LAUNCH_CHECK("k_scan_u32");
    }
    k_nodes<<<std::min(gn, 512u), 256, 0, st>>>(n, T->p.leaf_size, tb);
    TREVR_LAUNCH_CHECK("k_nodes");
    k_levels<<<std::min(gn, 512u), 256, 0, st>>>(n, tb);
    TREVR_LAUNCH_CHECK("k_levels");
    const unsigned gs = (unsigned)std::min<int64_t>(2 * n / kSubtree + 1, 8192);
    k_subtrees<<<gs, 256, 0, st>>>(n, B, nclass, linear, tb);
    TREVR_LAUNCH_CHECK("k_subtrees");
    hipError_t e = hipMemcpyAsync(T->host_u32, tb.levels,
                                  (2 * (kMaxLevels + 3) + kInfoWords) * sizeof(uint32_t),
                                  hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if ((rc = hip_check(e, "level readback")) != TREVR_OK) return rc;
    if (info[0] == 0u) break;
    if (wide) return set_error(TREVR_E_HIP, "the full sort did not finish");
    if ((rc = zero_words(st, &tb.words->resort, 1)) != TREVR_OK) return rc;
  }
  T->levels.clear();
  const uint2* lv = reinterpret_cast<const uint2*>(T->host_u32);
  for (uint32_t d = 0; d < info[2]; ++d) T->levels.emplace_back(lv[d].x, lv[d].y);
  T->num_nodes = info[1];
  T->num_leaves = (T->num_nodes + 1) / 2;
  T->depth = (int32_t)info[2];
  T->dev.num_nodes = T->num_nodes;
  T->dev.depth = T->depth;
  // the larger cells, deepest level first; the levels next to the root that
  // one workgroup takes in a step or two share a launch
  int one = 0;
  while (one < (int)info[3] &&
         (int64_t)(lv[one].y - lv[one].x) * (nclass * B + 1) <= 2 * 1024)
    ++one;
  for (int d = (int)info[3] - 1; d >= one; --d) {
    const int64_t work = (int64_t)(lv[d].y - lv[d].x) * (nclass * B + 1);
    k_cells<<<grid_for(work, 128), 128, 0, st>>>(d, d, B, nclass, linear, tb);
    TREVR_LAUNCH_CHECK("k_cells");
  }
  if (one > 0) {
    k_cells<<<1, 1024, 0, st>>>(one - 1, 0, B, nclass, linear, tb);
    TREVR_LAUNCH_CHECK("k_cells");
  }
  if (T->p.flags & TREVR_COMPLEX_SRC) {
    for (int d = T->depth - 1; d >= 0; --d) {
      const int64_t cw = (int64_t)(lv[d].y - lv[d].x) * T->nray;
      k_csrc<<<grid_for(cw, 128), 128, 0, st>>>(tb, lv[d].x, lv[d].y, B, nclass, T->nray);
      TREVR_LAUNCH_CHECK("k_csrc");
    }
  }
#undef TREVR_LAUNCH_CHECK
  // the kernels launched since the readback may still run when the call
  // returns: an event that calls on other streams wait for
  if (info[3] > 0u || (T->p.flags & TREVR_COMPLEX_SRC)) {
    hipError_t e = hipEventCreateWithFlags(&T->built, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventRecord(T->built, st);
    if ((rc = hip_check(e, "build event")) != TREVR_OK) return rc;
    T->building = true;
  }
  return TREVR_OK;
}

}  // namespace trevr
