// The mean-pool compression branch (Sec. 2 branch (i); Sec. 5.2 keeps it beside
// the covariance selector): per query head, softmax attention over the pooled
// blocks, block b entering as one key (its stored mean key) with one value (its
// stored mean value), over every block b < ceil(T/L).
//
// A workgroup of 16 waves takes HW query heads of one (batch row, KV head).
// Sixteen lanes share a block: lane ln owns elements [ln D/16, (ln+1) D/16) of
// its mean key and mean value, so a load instruction reads four whole vectors,
// the scores are 16-lane DPP sums that every lane of the group ends with, and
// the probabilities meet the values in the same lanes, with no LDS in the loop.
// A group takes four blocks at a time (all of their loads in flight, one rescale
// of its running state per head); the 64 groups' states merge in lane,
// then wave order.
//
// What bounds it: latency (the bytes of a case here, 17 MB for 4 x 8 units of
// 1024 blocks, are 3.5 us at the copy rate) and, with all heads of a large
// group in one workgroup, its CU's vector ALUs (2 G D multiply-adds per block).
// So the heads are split over workgroups until the chip is covered (see
// launch_compress); the workgroups of one unit read the same records, the
// later ones from L2.  10.5 us a call at that case (4 heads per KV head, bf16
// means; one 256-thread workgroup per unit, whose value pass loaded one block
// at a time, took 47.4).
#include "select_impl.h"

namespace cobs {

constexpr int kCmpThreads = 1024;

// Four floats of the queries, whose address need only be that of a float.
typedef float query4_t __attribute__((ext_vector_type(4), aligned(4)));

// Blocks of a 16-lane group per pass: two where four would spill (128 registers).
template <int D, int HW, int MDT>
constexpr int cmp_batch() { return (D == 128 && HW == 4 && MDT != DT_BF16) ? 2 : 4; }

// Elements [ln D/16, (ln+1) D/16) of a stored vector as raw words (E2M1 at
// D = 64: four codes, the low half word).
template <int D, int DT>
__device__ __forceinline__ void load_part(const uint8_t* vec, int ln, uint32_t* w) {
  constexpr int B = elem_bytes<DT>(D / 16);
  if constexpr (B >= 4) load_words<B / 4>(vec + ln * B, w);
  else w[0] = *reinterpret_cast<const uint16_t*>(vec + ln * B);
}

template <int D, int DT>
constexpr int part_words() { return elem_bytes<DT>(D / 16) >= 4 ? elem_bytes<DT>(D / 16) / 4 : 1; }

template <int D, int HW, int MDT>
__global__ __launch_bounds__(kCmpThreads) void compress_kernel(CompressParams p) {
  constexpr int EPL = D / 16, NW = kCmpThreads / 64, U = cmp_batch<D, HW, MDT>();
  constexpr int MW = part_words<D, MDT>();
  __shared__ float wm[NW][HW], wl[NW][HW];
  __shared__ __align__(16) float wo[NW][HW][D];

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int ln = lane & 15, grp = lane >> 4;
  // workgroups in runs of 8 units: the head splits of a unit are 8 indices
  // apart, on one XCD (its L2 serves all but the first) and dispatched together
  const int nsp = p.nsplit, run = 8 * nsp;
  const int unit = (int)(blockIdx.x / run) * 8 + (int)(blockIdx.x % 8), split = (int)(blockIdx.x % run) / 8;
  if (unit >= p.units) return;
  const int b = unit / p.hkv, h = unit % p.hkv;
  const int nb = blocks_of(clamp_len(p.seq_lens[b], p.tmax), p.lsh);
  const uint8_t* recu = p.rec + (int64_t)unit * p.nbmax * p.lay.total;
  const int64_t head0 = (int64_t)b * p.hq + (int64_t)h * (HW * nsp) + split * HW;

  float q[HW][EPL], m[HW], l[HW], o[HW][EPL];
#pragma unroll
  for (int g = 0; g < HW; ++g) {
    m[g] = -INFINITY;
    l[g] = 0.0f;
#pragma unroll
    for (int e = 0; e < EPL; e += 4) {
      const query4_t x = *reinterpret_cast<const query4_t*>(p.q + (head0 + g) * D + EPL * ln + e);
      q[g][e] = x.x * p.c; q[g][e + 1] = x.y * p.c; q[g][e + 2] = x.z * p.c; q[g][e + 3] = x.w * p.c;
    }
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[g][e] = 0.0f;
  }

  // Block base + 4 u + grp of pass element u; past the last block its record is
  // read again, its score is -inf and its value words are cleared (probability 0
  // times an infinite value would be NaN).  Only a wave's last pass can hold such
  // elements: the others are compiled without the tests.
  // With fp32 vectors of 128 elements and one head a pass's registers are loaded
  // for the next one as soon as they are unpacked (the keys before the softmax,
  // the values at the end of the pass): 4 x 8 units of 1016 blocks, two heads per
  // KV head, take 16.6 us instead of 20.3.  Smaller vectors gain nothing (bf16,
  // one head: 9.8 against 10.2 us ahead), and more heads leave no registers for it.
  constexpr int kStep = 4 * U * NW;
  constexpr bool kAhead = MDT == DT_F32 && D == 128 && HW == 1;
  uint32_t kw[U][MW], vw[U][MW];
  float ks[U], vs[U];
  auto load = [&](int base, auto keys, auto values) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint8_t* R = recu + (int64_t)min(base + 4 * u + grp, nb - 1) * p.lay.total;
      if constexpr (keys()) load_part<D, MDT>(R + p.lay.mean_off, ln, kw[u]);
      if constexpr (values()) load_part<D, MDT>(R + p.lay.vmean_off, ln, vw[u]);
      if constexpr (keys()) ks[u] = (MDT == DT_E2M1) ? *reinterpret_cast<const float*>(R + 4) : 1.0f;
      if constexpr (values()) vs[u] = (MDT == DT_E2M1) ? *reinterpret_cast<const float*>(R + 8) : 1.0f;
    }
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  if (kAhead && 4 * U * wave < nb) load(4 * U * wave, yes, yes);
  auto pass = [&](int base, auto whole) {
    const bool more = kAhead && base + kStep < nb;
    if constexpr (!kAhead) load(base, yes, yes);
    float sc[U][HW];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool live = whole() || base + 4 * u + grp < nb;
      // an infinite scale times its zero codes is NaN, and so is the score
      const float s = (MDT == DT_E2M1) ? __builtin_fmaf(ks[u], 0.0f, ks[u]) : 1.0f;
      float x[EPL];
      unpack_elems<MDT, EPL>(kw[u], x);
#pragma unroll
      for (int g = 0; g < HW; ++g) {
        float a = 0.0f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) a += x[e] * q[g][e];
        a = row16_sum(a) * s;
        sc[u][g] = live ? a : -INFINITY;
      }
    }
    if (more) load(base + kStep, yes, no);
#pragma unroll
    for (int g = 0; g < HW; ++g) {
      float mn = m[g];
#pragma unroll
      for (int u = 0; u < U; ++u) mn = fmaxf(mn, sc[u][g]);
      // (a group whose blocks all lie past the end keeps its empty state)
      const float ref = (mn == -INFINITY) ? 0.0f : mn;
      const float alpha = __expf(m[g] - ref);
      m[g] = mn;
      l[g] *= alpha;
#pragma unroll
      for (int e = 0; e < EPL; ++e) o[g][e] *= alpha;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        sc[u][g] = __expf(sc[u][g] - ref);
        l[g] += sc[u][g];
      }
    }
    if (!whole() && base + 4 * U > nb) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool live = base + 4 * u + grp < nb;
#pragma unroll
        for (int w = 0; w < MW; ++w) vw[u][w] = live ? vw[u][w] : 0u;
        vs[u] = live ? vs[u] : 0.0f;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float x[EPL];
      unpack_elems<MDT, EPL>(vw[u], x);
#pragma unroll
      for (int g = 0; g < HW; ++g) {
        const float pr = sc[u][g] * vs[u];
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[g][e] += pr * x[e];
      }
    }
    if (more) load(base + kStep, no, yes);
  };
  int base = 4 * U * wave;
  if constexpr (kAhead) {                // (two forms of the pass would spill)
    for (; base < nb; base += kStep) pass(base, no);
  } else {
    for (; base + 4 * U <= nb; base += kStep) pass(base, yes);
    if (base < nb) pass(base, no);
  }
  // ---- the four groups' states of the wave
#pragma unroll
  for (int k = 16; k < 64; k <<= 1) {
#pragma unroll
    for (int g = 0; g < HW; ++g) {
      const float m2 = __shfl_xor(m[g], k, 64), l2 = __shfl_xor(l[g], k, 64);
      const float mn = fmaxf(m[g], m2), ref = (mn == -INFINITY) ? 0.0f : mn;
      const float f1 = __expf(m[g] - ref), f2 = __expf(m2 - ref);
      m[g] = mn;
      l[g] = f1 * l[g] + f2 * l2;
#pragma unroll
      for (int e = 0; e < EPL; ++e) o[g][e] = f1 * o[g][e] + f2 * __shfl_xor(o[g][e], k, 64);
    }
  }
  if (grp == 0) {
#pragma unroll
    for (int g = 0; g < HW; ++g) {
      if (ln == 0) { wm[wave][g] = m[g]; wl[wave][g] = l[g]; }
#pragma unroll
      for (int e = 0; e < EPL; e += 4)
        *reinterpret_cast<float4*>(&wo[wave][g][EPL * ln + e]) = make_float4(o[g][e], o[g][e + 1], o[g][e + 2], o[g][e + 3]);
    }
  }
  __syncthreads();
  // ---- the waves' states, merged in wave order
  for (int idx = tid; idx < HW * D; idx += kCmpThreads) {
    const int g = idx / D, dd = idx % D;
    float M = -INFINITY;
#pragma unroll
    for (int k = 0; k < NW; ++k) M = fmaxf(M, wm[k][g]);
    float acc = 0.0f, lsum = 0.0f;
    if (M != -INFINITY) {
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const float f = __expf(wm[k][g] - M);
        acc += f * wo[k][g][dd];
        lsum += f * wl[k][g];
      }
    }
    const int64_t oq = head0 + g;
    p.out[oq * D + dd] = (lsum > 0.0f) ? acc / lsum : 0.0f;
    if (dd == 0 && p.lse) p.lse[oq] = (lsum > 0.0f) ? M + logf(lsum) : -INFINITY;
  }
}

typedef void (*CompressKernel)(CompressParams);

template <int D, int MDT>
static CompressKernel compress_kernel_h(int hw) {
  switch (hw) {
    case 1: return compress_kernel<D, 1, MDT>;
    case 2: return compress_kernel<D, 2, MDT>;
    default: return compress_kernel<D, 4, MDT>;
  }
}

template <int D>
static CompressKernel compress_kernel_m(int mdt, int hw) {
  if (mdt == DT_F32) return compress_kernel_h<D, DT_F32>(hw);
  if (mdt == DT_BF16) return compress_kernel_h<D, DT_BF16>(hw);
  return compress_kernel_h<D, DT_E2M1>(hw);
}

// Heads per workgroup: at most 4 (the queries and running outputs of more do
// not fit the 128 registers that 16 waves leave a lane), halved while the
// units alone leave CUs idle.
hipError_t launch_compress(CompressParams p, int d, int g, int batch, hipStream_t st) {
  const int64_t units = (int64_t)batch * p.hkv;
  int hw = std::min(g, 4);
  while (hw > 1 && units * (g / hw) < device_cus()) hw /= 2;
  p.units = (int)units;
  p.nsplit = g / hw;
  const CompressKernel k = (d == 128) ? compress_kernel_m<128>(p.mdt, hw) : compress_kernel_m<64>(p.mdt, hw);
  const int64_t grid = (units + 7) / 8 * 8 * p.nsplit;
  hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(kCmpThreads), 0, st, p);
  return hipGetLastError();
}

}  // namespace cobs
