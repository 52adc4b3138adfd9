// General path: any bucket size d (used for d > 8192, d = n among them, and for fixed width with d not a
// multiple of 4: decode of every such size, encode of those above 1024; the encoder of small buckets takes
// the others).
//
// Encode.  A bucket no longer fits one workgroup's registers, so it is cut into
// segments of 2048 values, one wavefront each, and the steps that the bucket path
// does inside a workgroup become kernels:
//   partial  sum of squares (fp64) or max of every group of up to sixteen segments -> workspace
//   scale    (buckets of several groups) their sum
//   encode   per-segment sub-stream (same wavefront code as the bucket path, with
//            code words wide enough for 32-bit gaps) -> workspace slot
//   scan     a workgroup per bucket walks its segments in order: which nonzero precedes a
//            segment's first one (max-scan), the bit offset of every segment in the
//            bucket string (sum-scan), the entry points
//   table    (several buckets) the word offset of every bucket; it, or `scan`, clears the
//            words that segments share
//   place    per segment: gap code, sub-stream and stop bit into the payload, shared words by OR
// Decode.  Records are added to a dense fp32 accumulator in the workspace, bucket by
// bucket and inside a bucket message after message (so every coordinate's sum has
// the order k = 0, 1, ...); a last kernel applies the accumulator to x.  Buckets
// above 8192 values carry a list of entry points behind their string and are read
// by a workgroup, a thread per stretch; shorter ones by a thread per bucket (levels
// above 127 only: the tile and split decoders take the others).
#include <cmath>

#include "qsgd_device.hpp"
#include "qsgd_encode_wave.hpp"
#include "qsgd_kernels.hpp"

namespace qsgd {

namespace {

constexpr int kSegChunks = 8;  // kSeg / kChunk

struct SegRef {
  uint64_t b;        // bucket
  uint32_t j;        // segment within the bucket
  uint64_t m;        // elements in the bucket
  uint32_t pos0;     // bucket position of the segment's first element
  uint32_t len;      // elements in the segment (0: past the end of a short bucket)
  uint64_t gidx0;    // global index of its first element
};

__device__ __forceinline__ SegRef seg_ref(const GenArgs& a, uint64_t seg) {
  SegRef r;
  r.b = seg / a.spb;
  r.j = (uint32_t)(seg - r.b * a.spb);
  const uint64_t base = r.b * a.d;
  r.m = min(a.d, a.n - base);
  const uint64_t p0 = (uint64_t)r.j * kSeg;
  r.pos0 = (uint32_t)p0;
  r.len = p0 < r.m ? (uint32_t)min((uint64_t)kSeg, r.m - p0) : 0u;
  r.gidx0 = base + p0;
  return r;
}

// Lane's four values of chunk c of a segment; any alignment, zeros past the end.
__device__ __forceinline__ float4 load_quad_any(const float* __restrict__ g, uint64_t gidx,
                                                uint32_t e, uint32_t len) {
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  const float* p = g + gidx + e;
  if (e + 3 < len && (((gidx + e) & 3u) == 0)) {
    v = *reinterpret_cast<const float4*>(p);
  } else {
    if (e + 0 < len) v.x = p[0];
    if (e + 1 < len) v.y = p[1];
    if (e + 2 < len) v.z = p[2];
    if (e + 3 < len) v.w = p[3];
  }
  return v;
}

}  // namespace

// ---- encode --------------------------------------------------------------------------

namespace {

// Segments of a bucket are added up in groups of G = 1, 2, 4, 8 or 16 (what a bucket has, or
// sixteen), a wavefront each; the groups of a bucket follow each other in `partial`.
constexpr uint32_t kPartialWaves = 16;
__host__ __device__ inline uint32_t group_size(uint64_t spb) { return spb >= 9 ? 16u : spb >= 5 ? 8u : spb >= 3 ? 4u : (uint32_t)spb; }
__host__ __device__ inline uint64_t groups_of(uint64_t spb) { const uint32_t G = group_size(spb); return (spb + G - 1) / G; }

}  // namespace

// Also writes the header and, fixed width, "no escape" into every bucket's string.  (13M values: 10 us,
// the bytes alone take 8 at the rate the card reads.)
__global__ __launch_bounds__(64 * kPartialWaves) void k_gen_partial(GenArgs a) {
  __shared__ double sums[kPartialWaves];
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    uint32_t* h = a.header;
    h[H_MAGIC] = kMagic; h[H_VERSION] = 1; h[H_CODE] = a.code; h[H_NORM] = a.norm_mode;
    h[H_S] = a.s; h[H_STREAM] = a.stream_id;
    h[H_D_LO] = (uint32_t)a.d; h[H_D_HI] = (uint32_t)(a.d >> 32);
    h[H_N_LO] = (uint32_t)a.n; h[H_N_HI] = (uint32_t)(a.n >> 32);
    h[H_NB_LO] = (uint32_t)a.nb; h[H_NB_HI] = (uint32_t)(a.nb >> 32);
    h[H_PW_LO] = (uint32_t)a.fixed_payload_words;
    h[H_PW_HI] = (uint32_t)(a.fixed_payload_words >> 32);
    h[H_STATUS] = 0; h[H_ITER] = a.iteration;
  }
  const uint32_t G = group_size(a.spb);
  const uint64_t gpb = groups_of(a.spb);
  const uint64_t group = (uint64_t)blockIdx.x * (kPartialWaves / G) + wave / G;
  const uint64_t b = group / gpb;
  const uint64_t j = (group - b * gpb) * G + wave % G;
  double ss = 0.0;
  if (b < a.nb && j < a.spb) {
    const SegRef r = seg_ref(a, b * a.spb + j);
    const float* const g = a.g + r.gidx0;
    float4 v[kSegChunks];
    if (r.len == kSeg) {
#pragma unroll
      for (int c = 0; c < kSegChunks; ++c) {
        const v4f_any x = *reinterpret_cast<const v4f_any*>(g + (uint32_t)c * kChunk + lane * 4u);
        v[c] = make_float4(x.x, x.y, x.z, x.w);
      }
    } else {
#pragma unroll
      for (int c = 0; c < kSegChunks; ++c)
        v[c] = load_quad_any(a.g, r.gidx0, (uint32_t)c * kChunk + lane * 4u, r.len);
    }
    if (a.norm_mode == 0) {
      double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
      for (int c = 0; c < kSegChunks; ++c) {
        s0 = fma((double)v[c].x, (double)v[c].x, s0);
        s1 = fma((double)v[c].y, (double)v[c].y, s1);
        s2 = fma((double)v[c].z, (double)v[c].z, s2);
        s3 = fma((double)v[c].w, (double)v[c].w, s3);
      }
      ss = wave_sum_f64((s0 + s1) + (s2 + s3));
    } else {
      float mx = 0.f;
#pragma unroll
      for (int c = 0; c < kSegChunks; ++c)
        mx = fmaxf(fmaxf(mx, fmaxf(fabsf(v[c].x), fabsf(v[c].y))), fmaxf(fabsf(v[c].z), fabsf(v[c].w)));
      ss = (double)wave_max_f32(mx);
    }
    if (j == 0 && a.code == QSGD_CODE_FIXED && lane == 0) a.payload[b * a.fixed_words_full + 1u] = 0xFFFFFFFFu;
  }
  if (lane == 0) sums[wave] = ss;
  __syncthreads();
  if (wave % G == 0 && lane == 0 && b < a.nb) {
    double t = sums[wave];
    for (uint32_t w = 1; w < G; ++w) t = a.norm_mode == 0 ? t + sums[wave + w] : fmax(t, sums[wave + w]);
    if (gpb == 1) a.scale[b] = a.norm_mode == 0 ? (float)sqrt(t) : (float)t;
    else a.partial[group] = t;
  }
}

// A workgroup per bucket adds up its groups.  (One wavefront took 7.6 us over the 6348 segments of 13M
// values.)
__global__ __launch_bounds__(256) void k_gen_scale(GenArgs a) {
  __shared__ double sums[4];
  const uint64_t b = blockIdx.x, n = groups_of(a.spb);
  const double* const p = a.partial + b * n;
  double acc = 0.0;   // (squares and magnitudes: 0 is below all of them)
  for (uint64_t g0 = threadIdx.x; g0 < n; g0 += 8 * 256) {
    double v[8];
#pragma unroll
    for (uint32_t t = 0; t < 8; ++t) v[t] = g0 + t * 256 < n ? p[g0 + t * 256] : 0.0;
#pragma unroll
    for (uint32_t t = 0; t < 8; ++t) acc = a.norm_mode == 0 ? acc + v[t] : fmax(acc, v[t]);
  }
  acc = a.norm_mode == 0 ? wave_sum_f64(acc) : (double)wave_max_f32((float)acc);
  if ((threadIdx.x & 63u) == 0) sums[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0)
    a.scale[b] = a.norm_mode == 0 ? (float)sqrt((sums[0] + sums[1]) + (sums[2] + sums[3]))
                                  : (float)fmax(fmax(sums[0], sums[1]), fmax(sums[2], sums[3]));
}

template <int CODE, bool ALIGNED>
__global__ __launch_bounds__(64) void k_gen_encode(GenArgs a) {
  extern __shared__ uint32_t smem[];
  uint32_t* const sub = smem;
  uint32_t* const ring = smem + a.sub_words;
  const int lane = threadIdx.x;
  const uint64_t seg = blockIdx.x;
  const SegRef r = seg_ref(a, seg);
  if (CODE != QSGD_CODE_FIXED) {
    for (uint32_t j = lane; j < a.sub_words; j += kWave) sub[j] = 0;
    __syncthreads();
  }
  WaveOut wo;
  wo.first_pos = 0; wo.last_pos = 0; wo.bits = 0;
  if (r.len) {
    float4 v[kSegChunks];
#pragma unroll
    for (int c = 0; c < kSegChunks; ++c) {
      v[c] = make_float4(0.f, 0.f, 0.f, 0.f);
      if ((uint32_t)c * kChunk < r.len)
        v[c] = load_quad_any(a.g, r.gidx0, (uint32_t)c * kChunk + lane * 4, r.len);
    }
    const float scale = a.scale[r.b];
    if (CODE == QSGD_CODE_FIXED && r.j == 0 && lane == 0) a.payload[r.b * a.fixed_words_full] = __float_as_uint(scale);
    QuantCtx qc;
    qc.s_f = (float)a.s;
    qc.inv = (scale > 0.f) ? qc.s_f / scale : 0.f;
    qc.s = a.s; qc.key0 = a.key0; qc.key1 = a.key1;
    qc.stream_id = a.stream_id; qc.iteration = a.iteration;
    const int nchunks = (int)((r.len + kChunk - 1) / kChunk);
    uint32_t rall[kSegChunks][4];
    draw_all<kSegChunks, ALIGNED>(a.index_base + r.gidx0, lane, qc, rall);
    if (CODE == QSGD_CODE_SPARSE) {
      encode_sparse_wave<kSegChunks, true>(v, rall, nchunks, r.pos0, lane, qc, ring, nullptr, sub, wo);
    } else if (CODE == QSGD_CODE_DENSE) {
      encode_dense_wave<kSegChunks>(v, rall, nchunks, r.len, lane, qc, sub, wo);
    } else {
      // fixed width: fields of 2048 values start on word boundaries in both planes
      const uint32_t B = a.fixed_bits, fmax = (1u << B) - 1u;
      uint32_t* const str = a.payload + r.b * a.fixed_words_full;
      const uint64_t lw = (r.m * B + 31) >> 5;
      uint32_t* const lplane = str + 2 + (((uint64_t)r.pos0 * B) >> 5);
      uint32_t* const splane = str + 2 + lw + (r.pos0 >> 5);
      const uint32_t lwn = (uint32_t)((r.len * B + 31u) >> 5), swn = (r.len + 31u) >> 5;
#pragma unroll
      for (int c = 0; c < kSegChunks; ++c) {
        if (c >= nchunks) break;
        const uint32_t e0 = (uint32_t)c * kChunk + lane * 4;
        const uint32_t (&rr)[4] = rall[c];
        const float vv[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
        uint32_t z[4], nib = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          z[j] = (e0 + j < r.len) ? quantize_one(vv[j], qc.inv, qc.s_f, qc.s, rr[j]) : 0u;
          if (z[j] > fmax) { str[1] = r.pos0 + e0 + j; z[j] = fmax; }
          nib |= (vv[j] < 0.f ? 1u : 0u) << j;
        }
        if (B == 8) {
          if ((e0 >> 2) < lwn) lplane[e0 >> 2] = z[0] | (z[1] << 8) | (z[2] << 16) | (z[3] << 24);
        } else if (B == 16) {
          if ((e0 >> 1) < lwn) lplane[e0 >> 1] = z[0] | (z[1] << 16);
          if ((e0 >> 1) + 1 < lwn) lplane[(e0 >> 1) + 1] = z[2] | (z[3] << 16);
        } else if (B == 4) {
          uint32_t h = z[0] | (z[1] << 4) | (z[2] << 8) | (z[3] << 12);
          h |= dpp_fetch<kDppShl1, 0xf>(h) << 16;
          if ((lane & 1) == 0 && (e0 >> 3) < lwn) lplane[e0 >> 3] = h;
        } else {
          uint32_t h = z[0] | (z[1] << 2) | (z[2] << 4) | (z[3] << 6);
          h |= dpp_fetch<kDppShl1, 0xf>(h) << 8;
          h |= dpp_fetch<kDppShl2, 0xf>(h) << 16;
          if ((lane & 3) == 0 && (e0 >> 4) < lwn) lplane[e0 >> 4] = h;
        }
        uint32_t sg = nib;
        sg |= dpp_fetch<kDppShl1, 0xf>(sg) << 4;
        sg |= dpp_fetch<kDppShl2, 0xf>(sg) << 8;
        sg |= dpp_fetch<kDppShl4, 0xf>(sg) << 16;
        if ((lane & 7) == 0 && (e0 >> 5) < swn) splane[e0 >> 5] = sg;
      }
    }
  }
  if (CODE == QSGD_CODE_FIXED) return;
  __syncthreads();
  if (lane == 0) {
    a.seginfo[seg] = wo.first_pos;
    a.seginfo[a.nseg + seg] = wo.last_pos;
    a.seginfo[2 * a.nseg + seg] = wo.bits;
  }
  uint32_t* slot = a.slots + seg * a.sub_words;
  const uint32_t nw = (wo.bits + 31u) >> 5;
  for (uint32_t j = lane; j < nw; j += kWave) slot[j] = sub[j];
}

// A workgroup walks a bucket's segments in order, kScanPer consecutive ones per thread and trip: a
// thread scans its own segments one after the other and the workgroup scans the threads' totals.
//
// Words of the payload that hold bits of two segments hold the first bit of one of them and the
// last bit of another: they are cleared (here if there is one bucket, else by `table`), and `place`
// ORs into them.  All other words have one writer.
//
// One bucket: latency and instruction issue of one compute unit.  6348 segments (13M values): 21.8 us
// with all buckets in one workgroup and 64-bit arithmetic throughout, and 4.7 for a launch that
// cleared the payload; 10 this way (eight segments per thread, one trip instead of two, or the second
// trip's loads ahead of the first: the same).
constexpr int kScanPer = 4;
typedef uint32_t v4u_any __attribute__((ext_vector_type(4), aligned(4)));

namespace {

// Bits of the recursive Elias code of k >= 1: groups of 1, 2, 3, 5, 9 and 17 bits or more.
__device__ __forceinline__ uint32_t omega_bits(uint32_t k) {
  const uint32_t n = 32u - (uint32_t)__clz((int)k);
  return n + (n > 1u ? 1u : 0u) + (n > 2u ? 2u : 0u) + (n > 4u ? 3u : 0u) + (n > 8u ? 1u : 0u) + (n > 16u ? 4u : 0u);
}

// Words [at, at + kScanPer) of an array of n (zeros past its end).
__device__ __forceinline__ void load_words(const uint32_t* p, uint64_t at, uint64_t n, uint32_t (&v)[kScanPer]) {
  if (at + kScanPer <= n) {
#pragma unroll
    for (int t = 0; t < kScanPer; t += 4) {
      const v4u_any x = *reinterpret_cast<const v4u_any*>(p + at + t);
      v[t] = x.x; v[t + 1] = x.y; v[t + 2] = x.z; v[t + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int t = 0; t < kScanPer; ++t) v[t] = at + t < n ? p[at + t] : 0u;
  }
}
__device__ __forceinline__ void store_words(uint32_t* p, uint64_t at, uint64_t n, const uint32_t (&v)[kScanPer]) {
  if (at + kScanPer <= n) {
#pragma unroll
    for (int t = 0; t < kScanPer; t += 4) {
      v4u_any x; x.x = v[t]; x.y = v[t + 1]; x.z = v[t + 2]; x.w = v[t + 3];
      *reinterpret_cast<v4u_any*>(p + at + t) = x;
    }
  } else {
#pragma unroll
    for (int t = 0; t < kScanPer; ++t) if (at + t < n) p[at + t] = v[t];
  }
}

// Inclusive scan over a workgroup of up to 16 wavefronts; `total`: of all of it.  The caller alternates
// between two buffers of wave totals: a barrier then lies between a buffer's reads and its next use.
template <bool MAX>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* wave_tot, uint32_t& total) {
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  v = MAX ? wave_incl_max_u32(v) : wave_incl_scan_u32(v, (int)lane);
  if (lane == 63u) wave_tot[wave] = v;
  __syncthreads();
  uint32_t pre = 0;
  total = 0;
  for (uint32_t w = 0; w < waves; ++w) {
    const uint32_t t = wave_tot[w];
    if (w == wave) pre = total;
    total = MAX ? max(total, t) : total + t;
  }
  return MAX ? max(pre, v) : pre + v;
}

// Clears the word of a bucket's string (at word `str` of the payload) in which a segment's bits end
// and others' may go on.  (The first segment with any starts on a word; the others start where one ends.)
__device__ __forceinline__ void clear_shared(const GenArgs& a, uint64_t str, uint64_t end, bool any) {
  if (any && (end & 31u) && str + (end >> 5) < a.cap_words) a.payload[str + (end >> 5)] = 0;
}

// Length and status of the message, and the table's padding.
__device__ __forceinline__ void close_message(const GenArgs& a, uint64_t total) {
  a.header[H_PW_LO] = (uint32_t)total;
  a.header[H_PW_HI] = (uint32_t)(total >> 32);
  for (uint64_t t = a.nb + 1; t < a.table_words; ++t) a.table[t] = 0;
  if (total > a.cap_words || total > 0xFFFFFFFFull) a.header[H_STATUS] = (uint32_t)QSGD_ERR_CAPACITY;
}

}  // namespace

__global__ __launch_bounds__(1024) void k_gen_scan(GenArgs a) {
  __shared__ uint32_t wave_tot[2][16], below[1024];
  const uint32_t tid = threadIdx.x, spb = (uint32_t)a.spb;
  const uint64_t b = blockIdx.x, base = b * a.spb;
  const uint64_t m = min(a.d, a.n - b * a.d);
  const uint32_t segs = (uint32_t)((m + kSeg - 1) / kSeg);   // (of spb: the last bucket has fewer)
  const bool sparse = a.code == QSGD_CODE_SPARSE;
  // of the trips before: last position, bits, entries, bits of the last segment
  uint32_t c_last = 0, c_ents = 0, c_tb = 0;
  uint64_t c_bits = 32;
  for (uint32_t s0 = 0; s0 < spb; s0 += kScanPer * blockDim.x) {
    const uint32_t j0 = s0 + tid * kScanPer;
    uint32_t first[kScanPer], last[kScanPer], bits[kScanPer];
    load_words(a.seginfo + base, j0, spb, first);
    load_words(a.seginfo + a.nseg + base, j0, spb, last);
    load_words(a.seginfo + 2 * a.nseg + base, j0, spb, bits);
    // which nonzero precedes each segment's first one: prefix maximum of the last positions
    uint32_t most = 0, total;
#pragma unroll
    for (int t = 0; t < kScanPer; ++t) most = first[t] ? last[t] : most;   // (they ascend)
    const uint32_t m_incl = block_scan<true>(most, wave_tot[0], total);
    const uint32_t m_below = dpp_fetch<kDppWaveShr1, 0xf>(m_incl);
    uint32_t prev[kScanPer], gap[kScanPer], tb[kScanPer];
    // (the thread below: of the same wavefront, or by way of LDS)
    uint32_t before = m_below;
    if ((tid & 63u) == 0) {
      before = 0;
      for (uint32_t w = 0; w < (tid >> 6); ++w) before = max(before, wave_tot[0][w]);
    }
    before = max(before, c_last);
    c_last = max(c_last, total);
    uint32_t sum = 0;
#pragma unroll
    for (int t = 0; t < kScanPer; ++t) {
      prev[t] = before;
      gap[t] = sparse && first[t] ? first[t] - before : 0u;
      before = first[t] ? last[t] : before;
      tb[t] = (gap[t] ? omega_bits(gap[t]) : 0u) + bits[t];   // (some 10^5 bits at most)
      sum += tb[t];
    }
    // bit offset of each segment inside its bucket string
    const uint32_t s_incl = block_scan<false>(sum, wave_tot[1], total);
    uint64_t start = c_bits + (s_incl - sum);
    c_bits += total;
    below[tid] = tb[kScanPer - 1];
    __syncthreads();
    const uint32_t tb_prev = tid ? below[tid - 1] : c_tb;
    // entry list: segment j >= 1 is listed iff its bit offset lies in a
    // later block of kEntryBits bits than the offset of segment j - 1
    static_assert(kEntryBits == 1024, "shift");
    uint32_t listed = 0;   // a bit per segment
    uint64_t at = start;
    uint32_t block = (uint32_t)((j0 ? start - tb_prev : start) >> 10);
#pragma unroll
    for (int t = 0; t < kScanPer; ++t) {
      const uint32_t now = (uint32_t)(at >> 10);
      listed |= now != block && j0 + t < segs && (at >> 32) == 0 ? 1u << t : 0u;
      block = now;
      at += tb[t];
    }
    c_tb = below[blockDim.x - 1];
    const uint32_t e_incl = block_scan<false>((uint32_t)__popc(listed), wave_tot[0], total);
    uint32_t rank = c_ents + e_incl - (uint32_t)__popc(listed);
    c_ents += total;
    uint32_t ranks[kScanPer];
#pragma unroll
    for (int t = 0; t < kScanPer; ++t) {
      ranks[t] = (listed >> t) & 1u ? rank : 0xFFFFFFFFu;
      rank += (listed >> t) & 1u;
      prev[t] = sparse ? prev[t] : (j0 + t) * kSeg;
    }
    at = start;
    if (j0 + kScanPer <= spb) {
      uint64_t* const out = a.segstart + base + j0;
#pragma unroll
      for (int t = 0; t < kScanPer; t += 2) {
        const uint64_t a1 = at + tb[t];
        v4u_any x; x.x = (uint32_t)at; x.y = (uint32_t)(at >> 32); x.z = (uint32_t)a1; x.w = (uint32_t)(a1 >> 32);
        *reinterpret_cast<v4u_any*>(out + t) = x;
        at = a1 + tb[t + 1];
      }
    } else {
#pragma unroll
      for (int t = 0; t < kScanPer; ++t) {
        if (j0 + t < spb) a.segstart[base + j0 + t] = at;
        at += tb[t];
      }
    }
    store_words(a.seggap + base, j0, spb, gap);
    store_words(a.segrank + base, j0, spb, ranks);
    store_words(a.segprev + base, j0, spb, prev);
    if (a.nb == 1) {
      at = start;
      if ((start + sum) >> 5 < a.cap_words) {
#pragma unroll
        for (int t = 0; t < kScanPer; ++t) {
          at += tb[t];
          if (tb[t] && ((uint32_t)at & 31u)) a.payload[at >> 5] = 0;
        }
      } else {
#pragma unroll 1
        for (int t = 0; t < kScanPer; ++t) {
          at += tb[t];
          clear_shared(a, 0, at, tb[t] != 0);
        }
      }
    }
    __syncthreads();
  }
  if (tid == 0) {
    const uint64_t words = ((c_bits + (sparse ? 1u : 0u) + 31u) >> 5) + 2ull * c_ents + 1u;
    a.bents[b] = c_ents;
    if (a.nb == 1) {
      a.table[0] = 0;
      a.table[1] = (uint32_t)min(words, (uint64_t)0xFFFFFFFFull);
      close_message(a, words);
    } else {
      a.words[b] = (uint32_t)min(words, (uint64_t)0xFFFFFFFFull);
    }
  }
}

// Several buckets: their word offsets, and the words that their segments share.  A workgroup takes a
// run of buckets and adds up the words of those before by itself.
__global__ __launch_bounds__(256) void k_gen_table(GenArgs a, uint32_t per) {
  __shared__ uint64_t part[4], str[256];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint64_t b_begin = (uint64_t)blockIdx.x * per, b_end = min(b_begin + per, a.nb);
  uint64_t base = 0;
#pragma unroll 8
  for (uint64_t b = tid; b < b_begin; b += 256) base += a.words[b];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) base += __shfl_xor(base, o, kWave);
  if (lane == 0) part[wave] = base;
  __syncthreads();
  base = (part[0] + part[1]) + (part[2] + part[3]);
  if (blockIdx.x == 0 && tid == 0) a.table[0] = 0;
  const uint32_t spb = (uint32_t)a.spb;
  for (uint64_t b0 = b_begin; b0 < b_end; b0 += 256) {
    const uint64_t b = b0 + tid;
    const uint64_t mine = b < b_end ? a.words[b] : 0u;
    uint64_t incl = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint64_t up = __shfl_up(incl, o, kWave);
      if (lane >= (uint32_t)o) incl += up;
    }
    __syncthreads();
    if (lane == 63u) part[wave] = incl;
    __syncthreads();
    uint64_t all = 0;
    for (uint32_t w = 0; w < 4; ++w) {
      if (w < wave) incl += part[w];
      all += part[w];
    }
    str[tid] = base + incl - mine;
    if (b < b_end) a.table[b + 1] = (uint32_t)min(base + incl, (uint64_t)0xFFFFFFFFull);
    __syncthreads();
    const uint32_t here = (uint32_t)min(b_end - b0, (uint64_t)256);
    for (uint32_t i = tid; i < here * spb; i += 256) {   // (spb is below 2^21: few buckets then)
      const uint64_t seg = b0 * spb + i;
      const uint32_t gap = a.seggap[seg];
      const uint32_t tb = (gap ? omega_bits(gap) : 0u) + a.seginfo[2 * a.nseg + seg];
      clear_shared(a, str[i / spb], a.segstart[seg] + tb, tb != 0);
    }
    base += all;
  }
  if (b_end == a.nb && tid == 0) close_message(a, base);
}

__global__ __launch_bounds__(256) void k_gen_place(GenArgs a) {
  if (a.header[H_STATUS] != 0) return;  // does not fit: nothing is written
  const uint32_t lane = threadIdx.x & 63u;
  const uint64_t seg = (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (seg >= a.nseg) return;
  const uint32_t bits = a.seginfo[2 * a.nseg + seg];
  const uint32_t gap = a.seggap[seg];
  const uint64_t start = a.segstart[seg];
  const uint32_t r = a.segrank[seg];
  const uint64_t b = seg / a.spb;
  const uint32_t j = (uint32_t)(seg - b * a.spb);
  uint32_t* const str = a.payload + a.table[b];
  uint64_t gc = 0;
  uint32_t glen = 0;
  if (gap) omega_encode(gap, gc, glen);
  const uint64_t end = start + glen + bits;
  if (lane == 0) {
    if (j == 0) str[0] = __float_as_uint(a.scale[b]);
    if (j == a.spb - 1 && a.code == QSGD_CODE_SPARSE) {   // the stop bit
      if (end & 31u) atomicOr(&str[end >> 5], 0x80000000u >> (end & 31u));
      else str[end >> 5] = 0x80000000u;
    }
    // the entry list sits behind the string's last word: pairs, then their count
    const uint32_t ents = a.bents[b];
    uint32_t* const list = a.payload + a.table[b + 1] - (2u * ents + 1u);
    if (r != 0xFFFFFFFFu) {
      list[2u * r] = (uint32_t)start;
      list[2u * r + 1u] = a.segprev[seg];
    }
    if (j == a.spb - 1) list[2u * ents] = ents;
  }
  if (end == start) return;
  // word i of the segment's words: the gap's code word (at the top of `top`), then the slot's bits
  const uint64_t top = glen ? gc << (64u - glen) : 0ull;
  const uint32_t sh = (uint32_t)(start & 31u), off = sh + glen;
  uint32_t* const out = str + (start >> 5);
  const uint32_t words = (uint32_t)(((end + 31u) >> 5) - (start >> 5));
  const uint32_t* const slot = a.slots + seg * a.sub_words;
  const uint32_t nw = (bits + 31u) >> 5;
  for (uint32_t i = lane; i < words; i += kWave) {
    uint32_t x = i == 0 ? (uint32_t)(top >> 32 >> sh)
               : i == 1 ? (uint32_t)(top >> sh)
               : i == 2 && sh ? (uint32_t)top << (32u - sh) : 0u;
    const int32_t rel = (int32_t)(32u * i - off);   // slot bit at the word's first bit
    const int32_t q = rel >> 5;
    const uint32_t lo = q >= 0 && (uint32_t)q < nw ? slot[q] : 0u;
    const uint32_t hi = q + 1 >= 0 && (uint32_t)(q + 1) < nw ? slot[q + 1] : 0u;
    x |= (uint32_t)(((uint64_t)lo << 32 | hi) << (rel & 31) >> 32);
    const bool shared = (i == 0 && sh) || (i == words - 1u && (end & 31u));
    if (shared) atomicOr(&out[i], x);
    else out[i] = x;
  }
}

// ---- decode --------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_gen_zero(float* p, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256)
    p[i] = 0.f;
}

// Four consecutive words of a string in registers (zeros past its end): three serve a
// 64-bit peek at any bit offset of the first one, the fourth is requested one word
// ahead of its use so that a reader does not wait for memory at every record.
struct WordWindow {
  const uint32_t* str;
  uint64_t nwords, wi;   // w0..w3 = words wi..wi+3
  uint32_t w0, w1, w2, w3;
  __device__ __forceinline__ uint32_t word(uint64_t i) const { return i < nwords ? str[i] : 0u; }
  __device__ __forceinline__ void open(const uint32_t* s, uint64_t n, uint64_t bitpos) {
    str = s; nwords = n; wi = bitpos >> 5;
    w0 = word(wi); w1 = word(wi + 1); w2 = word(wi + 2); w3 = word(wi + 3);
  }
  // The 64 stream bits from `bitpos` on; bitpos never moves backwards.
  __device__ __forceinline__ uint64_t peek(uint64_t bitpos) {
    while (wi < (bitpos >> 5)) {
      w0 = w1; w1 = w2; w2 = w3;
      w3 = word(wi + 4);
      ++wi;
    }
    const uint32_t off = (uint32_t)(bitpos & 31u);
    const uint64_t hi = ((uint64_t)w0 << 32) | w1;
    return off ? (hi << off) | (w2 >> (32u - off)) : hi;
  }
};

// One string, read front to back from (bitpos, pos) until `stop` (or, for the last
// stretch of a Code'_s string, until position m); values are ADDED to out[] with plain
// read-modify-writes: the caller guarantees that nobody else touches this bucket's
// part of out[] at the same time.  Returns false on malformed input.
__device__ __forceinline__ bool parse_stretch(const uint32_t* str, uint64_t nwords, bool sparse,
                                              bool to_end_of_bucket, uint64_t stop, uint64_t m,
                                              uint32_t s, float scale, uint64_t& bitpos,
                                              uint64_t& pos, float* out) {
  WordWindow win;
  win.open(str, nwords, bitpos);
  // Records are read kBatch at a time and then added together: the additions of one
  // message hit distinct coordinates, so their loads can all be in flight at once
  // instead of one memory round trip per record.
  constexpr int kBatch = 8;
  for (;;) {
    float* where[kBatch];
    float what[kBatch];
    bool done = false;
#pragma unroll
    for (int t = 0; t < kBatch; ++t) {
      where[t] = nullptr;
      what[t] = 0.f;
      if (done) continue;
      if (to_end_of_bucket ? pos >= m : bitpos >= stop) { done = true; continue; }
      uint32_t gl = 0, gap = 1;
      if (sparse) {
        gap = omega_loop(win.peek(bitpos), gl);
        if (gap == 0) return false;
      }
      const uint64_t w = win.peek(bitpos + gl);
      uint32_t ll;
      uint32_t lev = omega_loop(w << 1, ll);
      bitpos += gl + 1u + ll;
      pos += gap;
      if (lev == 0 || pos > m || bitpos > stop) return false;
      if (!sparse) lev -= 1u;
      if (lev > s) return false;
      if (lev) {
        const float mag = scale * (float)lev;
        where[t] = out + (pos - 1);
        what[t] = (w >> 63) ? -mag : mag;
      }
    }
    float old[kBatch];
#pragma unroll
    for (int t = 0; t < kBatch; ++t) old[t] = where[t] ? *where[t] : 0.f;
#pragma unroll
    for (int t = 0; t < kBatch; ++t)
      if (where[t]) *where[t] = old[t] + what[t];
    if (done) return true;
  }
}

// Where a bucket string of message k lies and where its records end.
struct StringRef {
  const uint32_t* str;
  uint64_t nwords;   // words of the string proper
  uint64_t endbit;   // records end here
  const uint32_t* list;
  uint64_t ents;     // entry points behind the string
  float scale;
};

__device__ __forceinline__ bool open_string(const DecodeArgs& a, uint32_t k, uint64_t b,
                                            bool entries, StringRef& r) {
  const uint32_t* msg = a.msgs[k];
  const uint64_t pay = (uint64_t)H_WORDS + a.table_words;
  const uint32_t o0 = msg[H_WORDS + b], o1 = msg[H_WORDS + b + 1];
  if (!(o0 < o1 && pay + o1 <= a.msg_words[k])) return false;
  r.str = msg + pay + o0;
  uint64_t words = o1 - o0;
  r.ents = 0;
  r.list = nullptr;
  if (entries) {
    r.ents = r.str[words - 1];
    if (2 * r.ents + 1 >= words) return false;
    words -= 2 * r.ents + 1;
    r.list = r.str + words;
  }
  r.nwords = words;
  r.scale = __uint_as_float(r.str[0]) / (float)a.s;
  r.endbit = words * 32;
  if (a.code == QSGD_CODE_SPARSE) {
    const uint32_t last = r.str[words - 1];
    if (last == 0) return false;
    r.endbit = words * 32 - 1 - (uint32_t)(__ffs((int)last) - 1);
    if (r.endbit < 32) return false;
  }
  return true;
}

// Short buckets of the general path (d <= kEntryMinD, d not a multiple of 4, s > 127): one thread
// per bucket reads the K strings one after the other, so every coordinate receives its
// terms in message order.
__global__ __launch_bounds__(256) void k_gen_parse(DecodeArgs a, float* acc) {
  if (*a.status != 0) return;
  const uint64_t b = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (b >= a.nb) return;
  const uint64_t base = b * (uint64_t)a.d;
  const uint64_t m = min((uint64_t)a.d, a.n - base);
  const bool sparse = a.code == QSGD_CODE_SPARSE;
  for (uint32_t k = 0; k < a.K; ++k) {
    StringRef r;
    if (!open_string(a, k, b, false, r)) { flag_corrupt(a.status); return; }
    uint64_t bitpos = 32, pos = 0;
    if (!parse_stretch(r.str, r.nwords, sparse, !sparse, r.endbit, m, a.s, r.scale, bitpos, pos,
                       acc + base) ||
        (!sparse && bitpos > r.endbit)) {
      flag_corrupt(a.status);
      return;
    }
  }
}

// Opens the K strings of bucket b side by side (a chain of dependent reads each).
// Returns false (every thread) if one of them is malformed.  Ends with a barrier.
__device__ __forceinline__ bool open_strings(const DecodeArgs& a, uint64_t b, StringRef* refs,
                                             uint32_t* bad) {
  if (threadIdx.x < a.K) {
    StringRef mine;
    if (open_string(a, threadIdx.x, b, true, mine)) refs[threadIdx.x] = mine;
    else *bad = 1;
  }
  __syncthreads();
  return *bad == 0;
}

// The messages take their turns (a barrier in between), a thread per stretch between two
// entry points: every coordinate receives its terms in message order.  Every stretch must
// end exactly where the next one starts, at the position the list names.
__device__ __forceinline__ bool parse_in_turns(const DecodeArgs& a, const StringRef* refs,
                                               uint64_t m, float* out, uint32_t* bad) {
  const bool sparse = a.code == QSGD_CODE_SPARSE;
  for (uint32_t k = 0; k < a.K; ++k) {
    const StringRef sr = refs[k];
    int my_bad = 0;
    for (uint64_t r = threadIdx.x; r <= sr.ents; r += blockDim.x) {
      uint64_t bitpos = r ? sr.list[2 * (r - 1)] : 32;
      uint64_t pos = r ? sr.list[2 * (r - 1) + 1] : 0;
      const bool last_stretch = r == sr.ents;
      const uint64_t stop = last_stretch ? sr.endbit : sr.list[2 * r];
      bool ok = bitpos >= 32 && bitpos <= stop && stop <= sr.endbit && pos <= m;
      ok = ok && parse_stretch(sr.str, sr.nwords, sparse, last_stretch && !sparse, stop, m, a.s,
                               sr.scale, bitpos, pos, out);
      // the stretch ends where the next one starts, at the position the list names
      if (ok && !last_stretch) ok = bitpos == stop && pos == sr.list[2 * r + 1];
      if (ok && last_stretch && !sparse) ok = pos == m && bitpos <= sr.endbit;
      if (!ok) my_bad = 1;
    }
    // message k is in before message k + 1 adds to the same coordinates; the barrier also
    // carries the verdict, so that every thread leaves (or stays) together
    if (__syncthreads_or(my_bad)) {
      if (threadIdx.x == 0) *bad = 1;
      return false;
    }
  }
  return true;
}

// Long buckets (d > kEntryMinD): the string is followed by a list of entry points, so a
// workgroup reads one bucket with a thread per stretch, message after message.
__global__ __launch_bounds__(256) void k_gen_parse_entries(DecodeArgs a, float* acc) {
  if (damaged_before(a.status)) return;
  __shared__ uint32_t bad;
  __shared__ StringRef refs[QSGD_MAX_PEERS];
  if (threadIdx.x == 0) bad = 0;
  const uint64_t b = blockIdx.x;
  const uint64_t base = b * (uint64_t)a.d;
  const uint64_t m = min((uint64_t)a.d, a.n - base);
  __syncthreads();
  if (!open_strings(a, b, refs, &bad) || !parse_in_turns(a, refs, m, acc + base, &bad)) {
    if (threadIdx.x == 0) flag_corrupt(a.status);
  }
}

// ---- long buckets of sparse Code_s messages ------------------------------------------------
// Where the host expects few coordinates that several messages hit, nearly all of x stays as it
// is, so no dense accumulator is made: the records of all K messages are listed first (a
// damaged message must leave x alone), then each updates its own coordinate.  Four launches:
//   clear    checks the headers, clears the bucket's bitmaps and counters
//   list     a workgroup per stretch between entry points: (position, value) into the message's
//            list, the position's bit into `seen` and, if it was set already, into `multi`
//   apply    a record whose position is not in `multi` updates x (0 + v is the sum in message
//            order), the others go to the bucket's collision list
//   resolve  a coordinate on that list is summed from 0 in message order by the thread that
//            holds its record of the lowest message.  Where the messages collide more often
//            than that list has room for, every coordinate in `multi` gets an accumulator
//            instead, and the messages' lists are gone through one after the other; where
//            a message's own list overflowed, the bucket's workgroup reads the messages in
//            turns into a dense accumulator.  Both are linear in the number of records.
// Bound by latency and four launches.  13M values, s = 1, K = 16: 180 us with a dense accumulator (zeroed,
// counted, stored, resolved, applied: 24 us of it for x alone), 46 with a thread per stretch, record
// after record (46 of them, 0.65 us each), 30 with a lane per bit (of the list's 15: 2 to open the
// string, 5 for the bits, 1 for a dozen rounds, 4 for the atomics); 13M values, d = 9000, s = 2, K = 8,
// where a wavefront had two stretches, 640 and 190.  Workgroups of two or eight wavefronts: list 17
// and 16 instead of 15 us, 124 and 234 instead of 124.
// Untouched coordinates: fma(-c, 0, x) is x for c >= 0; where it is not (accumulating, and
// c < 0, turn -0 into +0) one more launch does that.

struct CollideList {
  uint32_t* count;
  uint32_t* overflow;   // the records did not fit: the messages are read in turns
  uint32_t* pos;
  float* val;
  uint32_t* msg;
};
__device__ __forceinline__ CollideList collide_list(uint8_t* lists, uint64_t b) {
  uint8_t* const base = lists + b * (uint64_t)kCollideBytes;
  CollideList l;
  l.count = reinterpret_cast<uint32_t*>(base);
  l.overflow = l.count + 1;
  l.pos = reinterpret_cast<uint32_t*>(base + 256);
  l.val = reinterpret_cast<float*>(base + 256 + 4 * kCollide);
  l.msg = reinterpret_cast<uint32_t*>(base + 256 + 8 * kCollide);
  return l;
}

// A bucket's share of the accumulator area, m words: two bitmaps, a counter per message, the
// messages' lists of records (two words each), and an accumulator for every coordinate that two
// messages can name (half as many as there are records).  cap 0: too small a bucket for that.
__host__ __device__ constexpr uint32_t bitmap_words(uint32_t m) { return (m >> 5) + (m % 32u ? 1u : 0u); }   // (m + 31 can overflow)
struct SparseArea {
  uint32_t *seen, *multi, *count;
  uint32_t fixed;   // words in front of the lists
  uint32_t cap;     // records per list
  uint32_t* lists;
  float* sums;      // K * cap / 2
  __device__ uint32_t* pos(uint32_t k) const { return lists + 2ull * k * cap; }
  __device__ uint32_t* val(uint32_t k) const { return lists + (2ull * k + 1ull) * cap; }
};
__device__ __forceinline__ SparseArea sparse_area(uint32_t* area, uint64_t base, uint32_t m,
                                                  uint32_t K) {
  SparseArea s;
  const uint32_t mw = bitmap_words(m);
  s.seen = area + base;
  s.multi = s.seen + mw;
  s.count = s.multi + mw;
  s.fixed = 2u * mw + K;
  s.lists = s.seen + s.fixed;
  s.cap = m > s.fixed ? (uint32_t)(2ull * (m - s.fixed) / (5u * K)) : 0u;
  s.sums = reinterpret_cast<float*>(s.lists + 2ull * K * s.cap);
  return s;
}

__global__ __launch_bounds__(256) void k_sparse_clear(DecodeArgs a, uint32_t* area, uint8_t* lists) {
  if (blockIdx.x == 0) check_headers(a);
  const uint32_t per = 2u * bitmap_words(a.d) + a.K;   // words of a full bucket
  const uint64_t total = (uint64_t)a.nb * per;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < total;
       i += (uint64_t)gridDim.x * 256) {
    const uint32_t b = (uint32_t)(i / per), w = (uint32_t)(i - (uint64_t)b * per);
    const uint64_t base = (uint64_t)b * a.d;
    const uint32_t m = (uint32_t)min((uint64_t)a.d, a.n - base);
    const SparseArea s = sparse_area(area, base, m, a.K);
    if (w == 0) {
      const CollideList cl = collide_list(lists, b);
      *cl.count = 0;
      *cl.overflow = s.cap ? 0u : 1u;
    }
    if (s.cap && w < s.fixed) s.seen[w] = 0;
  }
}

// A workgroup per stretch, kListWords words of it at a time.  Nobody reads record after record: a lane
// for every BIT reads the record that would begin there (all of them side by side), four rounds of
// "where does the record at my end lead" give every word a table of where one leaves it from each of
// its bits, and a lane per word follows those tables from the stretch's start, which is known, until
// no word's entry changes any more.
constexpr uint32_t kListWords = 64, kListThreads = 256;
__global__ __launch_bounds__(kListThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_sparse_list(DecodeArgs a, uint32_t* area, uint8_t* lists) {
  if (damaged_before(a.status)) return;
  __shared__ uint32_t words[kListWords + 4], what[kListWords * 32], gaps[kListWords * 32], carry[2];
  __shared__ uint8_t leaves[kListWords * 32];
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t b = blockIdx.x;
  const uint32_t k = blockIdx.y;
  StringRef sr;
  if (!open_string(a, k, b, true, sr)) {   // (the same in every lane)
    if (tid == 0) flag_corrupt(a.status);
    return;
  }
  const uint64_t base = b * (uint64_t)a.d;
  const uint32_t m = (uint32_t)min((uint64_t)a.d, a.n - base);
  const SparseArea s = sparse_area(area, base, m, a.K);
  uint32_t* const lpos = s.pos(k);
  uint32_t* const lval = s.val(k);
  uint32_t* const overflow = collide_list(lists, b).overflow;

  for (uint64_t r = blockIdx.z; r <= sr.ents; r += gridDim.z) {
    const bool last_stretch = r == sr.ents;
    const uint64_t bitpos = r ? sr.list[2 * (r - 1)] : 32;
    const uint64_t stop = last_stretch ? sr.endbit : sr.list[2 * r];
    const uint32_t pos_end = last_stretch ? 0u : sr.list[2 * r + 1];
    uint32_t at_pos = r ? sr.list[2 * (r - 1) + 1] : 0u;
    if (!(bitpos >= 32 && bitpos <= stop && stop <= sr.endbit && at_pos <= m) ||
        (bitpos == stop && !last_stretch && at_pos != pos_end)) {
      if (tid == 0) flag_corrupt(a.status);
      continue;
    }
    uint32_t entry0 = (uint32_t)(bitpos & 31u);
    for (uint64_t w0 = bitpos >> 5; w0 * 32u < stop; w0 += kListWords) {
      const uint32_t here = (uint32_t)min((uint64_t)kListWords, ((stop + 31u) >> 5) - w0);
      if (tid < here + 4u) words[tid] = w0 + tid < sr.nwords ? sr.str[w0 + tid] : 0u;
      __syncthreads();
      for (uint32_t t0 = 2u * wave; t0 < here; t0 += kListThreads / 32u) {
        const uint32_t t = t0 + (lane >> 5), o = lane & 31u;   // (t may be `here`: nobody asks for it)
        const uint32_t x0 = words[t], x1 = words[t + 1u], x2 = words[t + 2u], x3 = words[t + 3u];
        const uint32_t h0 = x0 >> 1, h1 = __builtin_amdgcn_alignbit(x0, x1, 1);
        const uint32_t h2 = __builtin_amdgcn_alignbit(x1, x2, 1), h3 = __builtin_amdgcn_alignbit(x2, x3, 1);
        // 32 bits from bit q on, q < 96
        auto peek = [&](uint32_t q) {
          const bool one = q >= 32u, two = q >= 64u;
          uint32_t hi = one ? h1 : h0, lo = one ? h2 : h1;
          hi = two ? h2 : hi;
          lo = two ? h3 : lo;
          return __builtin_amdgcn_alignbit(hi, lo, ~q);
        };
        uint32_t gl, ll, open, more;
        const uint32_t v = peek(o);
        uint32_t gap = by_last_group(v, last_group_bits(v), gl, open);
        if (open) {
          // four groups, of 2, 3, 5 and gap + 1 bits (2^16 to 2^32 - 1), or malformed
          more = gap;
          const bool four = more >= 16u && more <= 31u && peek(o + 11u + (more & 31u)) >> 31 == 0;
          gap = four ? peek(o + 10u) >> (31u - (more & 31u)) : 0u;
          gl = (more & 31u) + 12u;                             // (43 at most)
        }
        const uint32_t w = peek(o + gl);
        const uint32_t lev = by_last_group(w << 1, last_group_bits(w << 1), ll, open);
        const bool good = gap != 0 && gap <= m && !open && lev <= a.s;
        const uint32_t len = gl + 1u + ll;                     // (67 at most)
        uint32_t to = good ? o + len : 32u;
        what[t * 32u + o] = good ? len | (w >> 31) << 7 | lev << 8 : 0u;   // length, sign, level
        gaps[t * 32u + o] = gap;
#pragma unroll
        for (int i = 0; i < 4; ++i) {                          // (eleven records at most in a word)
          const uint32_t on = (uint32_t)__shfl((int)to, (int)((lane & 32u) | (to & 31u)), kWave);
          to = to < 32u ? on : to;
        }
        leaves[t * 32u + o] = (uint8_t)to;
      }
      __syncthreads();
      if (wave == 0) {
        const uint64_t word_bit = (w0 + lane) * 32u;
        const uint32_t end = lane < here && word_bit < stop ? (uint32_t)min((uint64_t)32, stop - word_bit) : 0u;
        const bool idle = end == 0;
        uint32_t entry = lane == 0 ? entry0 : 0u, exit = 0;
        bool again = !idle;
        for (uint32_t round = 0; round <= kListWords; ++round) {
          if (again) exit = entry < 32u ? leaves[lane * 32u + entry] : entry;
          const uint32_t below = (uint32_t)__shfl_up((int)exit, 1, kWave) - 32u;
          const uint32_t now = lane == 0 || idle ? entry : below;
          again = now != entry;
          entry = now;
          if (__builtin_amdgcn_ballot_w64(again) == 0) break;
        }
        // the word's records
        constexpr int kMost = 11;
        uint32_t rec[kMost], gap[kMost], o = entry, adv = 0;
        bool ok = true;
#pragma unroll
        for (int i = 0; i < kMost; ++i) {
          rec[i] = gap[i] = 0;
          if (o < end && ok) {
            rec[i] = what[lane * 32u + o];
            gap[i] = gaps[lane * 32u + o];
            ok = rec[i] != 0;
            if (ok) { adv += gap[i]; o += rec[i] & 127u; }
          }
        }
        const uint32_t p_incl = wave_incl_scan_u32(adv, (int)lane);
        uint32_t p = at_pos + p_incl - adv;
        // (not the new position <= m: it is counted in 32 bits and could come round)
        uint32_t sound = 0;
#pragma unroll
        for (int i = 0; i < kMost; ++i) {
          if (rec[i]) {
            ok = ok && p <= m && gap[i] <= m - p;
            p += gap[i];
            gap[i] = p - 1u;                                   // (the record's place from here on)
            sound += ok ? 1u : 0u;
          }
        }
        // the stretch ends where the next one starts, at the position the list names
        const bool final_word = !idle && word_bit + 32u >= stop;
        if (!idle && (!ok || (final_word && (o != end || (!last_stretch && p != pos_end))))) flag_corrupt(a.status);
        // deliver: a place in the message's list for every record, and its bit
        const uint32_t incl = wave_incl_scan_u32(sound, (int)lane);
        const uint32_t total = lane_bcast(incl, 63);
        uint32_t at = 0;
        if (s.cap && lane == 0 && total) at = atomicAdd(&s.count[k], total);
        at = lane_bcast(at, 0);
        if (at + total > s.cap) {
          if (lane == 0) *overflow = 1;
        } else {
          at += incl - sound;
          uint32_t old[kMost];
#pragma unroll
          for (int i = 0; i < kMost; ++i) {
            old[i] = 0;
            if ((uint32_t)i < sound) {
              const float mag = sr.scale * (float)(rec[i] >> 8);
              old[i] = atomicOr(&s.seen[gap[i] >> 5], 1u << (gap[i] & 31u));
              lpos[at + i] = gap[i];
              lval[at + i] = __float_as_uint((rec[i] >> 7) & 1u ? -mag : mag);
            }
          }
#pragma unroll
          for (int i = 0; i < kMost; ++i) {
            if ((uint32_t)i < sound && (old[i] >> (gap[i] & 31u)) & 1u)
              atomicOr(&s.multi[gap[i] >> 5], 1u << (gap[i] & 31u));
          }
        }
        // what the next words go on from
        if (lane == kListWords - 1u) { carry[0] = exit - 32u; carry[1] = at_pos + p_incl; }
      }
      __syncthreads();
      if (here == kListWords) { entry0 = carry[0]; at_pos = carry[1]; }
    }
  }
}

__device__ __forceinline__ float updated(const DecodeArgs& a, float x, float sum) {
  return a.step ? fmaf(-a.c, sum, x) : x + sum;
}

__global__ __launch_bounds__(256) void k_sparse_apply(DecodeArgs a, uint32_t* area, uint8_t* lists) {
  if (*a.status != 0) return;
  const uint64_t b = blockIdx.x;
  const uint32_t k = blockIdx.y;
  const CollideList cl = collide_list(lists, b);
  if (*cl.overflow) return;
  const uint64_t base = b * (uint64_t)a.d;
  const uint32_t m = (uint32_t)min((uint64_t)a.d, a.n - base);
  const SparseArea s = sparse_area(area, base, m, a.K);
  const uint32_t n = s.count[k];
  const uint32_t* const lpos = s.pos(k);
  const uint32_t* const lval = s.val(k);
  float* const x = a.x + base;
  constexpr uint32_t kU = 2;
  const uint32_t step = 256u * gridDim.z;
  for (uint32_t i0 = blockIdx.z * 256u + threadIdx.x; i0 < n; i0 += kU * step) {
    uint32_t p[kU], bits[kU];
    float v[kU], old[kU];
#pragma unroll
    for (uint32_t j = 0; j < kU; ++j) {
      const uint32_t i = min(i0 + j * step, n - 1u);
      p[j] = lpos[i];
      v[j] = __uint_as_float(lval[i]);
    }
#pragma unroll
    for (uint32_t j = 0; j < kU; ++j) { bits[j] = s.multi[p[j] >> 5]; old[j] = x[p[j]]; }
#pragma unroll
    for (uint32_t j = 0; j < kU; ++j) {
      if (i0 + j * step >= n) continue;
      if (((bits[j] >> (p[j] & 31u)) & 1u) == 0) {   // (only this record names the coordinate)
        x[p[j]] = updated(a, old[j], 0.f + v[j]);    // (a sum starts from +0: -0 does not stay)
      } else {
        const uint32_t idx = atomicAdd(cl.count, 1u);
        if (idx < kCollide) { cl.pos[idx] = p[j]; cl.val[idx] = v[j]; cl.msg[idx] = k; }
      }
    }
  }
}

__global__ __launch_bounds__(1024) void k_sparse_resolve(DecodeArgs a, uint32_t* area, uint8_t* lists) {
  if (damaged_before(a.status)) return;
  __shared__ uint32_t bad;
  __shared__ StringRef refs[QSGD_MAX_PEERS];
  __shared__ uint32_t lpos[kCollide];
  __shared__ float lval[kCollide];
  __shared__ uint8_t lk[kCollide];
  constexpr int kHashBits = 11;
  __shared__ uint32_t head[1 << kHashBits], next[kCollide];
  __shared__ uint32_t wave_total[1024 / 64];
  const uint64_t b = blockIdx.x;
  const uint64_t base = b * (uint64_t)a.d;
  const uint32_t m = (uint32_t)min((uint64_t)a.d, a.n - base);
  float* const x = a.x + base;
  for (uint32_t i = threadIdx.x; i < (1u << kHashBits); i += blockDim.x) head[i] = 0xFFFFFFFFu;
  const CollideList cl = collide_list(lists, b);
  const bool overflow = *cl.overflow != 0;
  const uint32_t L = *cl.count;
  if (overflow || L > kCollide) {
    // (the messages parsed before; coordinates that `apply` has updated already are told by
    // their bits, before the area becomes the accumulator)
    const SparseArea s = sparse_area(area, base, m, a.K);
    float* const acc = reinterpret_cast<float*>(area) + base;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    if (!overflow) {
      // the collision list alone was too short: the coordinates in `multi` remain.  `seen` has
      // done its work and takes the number of them before every word of the bitmap.
      const uint32_t mw = bitmap_words(m), lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
      constexpr uint32_t kPer = 8;   // words per thread and trip
      uint32_t before = 0;
      for (uint32_t w0 = 0; w0 < mw; w0 += 1024u * kPer) {
        const uint32_t at = w0 + threadIdx.x * kPer;
        uint32_t cnt[kPer], mine = 0;
#pragma unroll
        for (uint32_t j = 0; j < kPer; ++j) {
          cnt[j] = at + j < mw ? (uint32_t)__popc(s.multi[at + j]) : 0u;
          mine += cnt[j];
        }
        const uint32_t incl = wave_incl_scan_u32(mine, (int)lane);
        if (lane == 63u) wave_total[wave] = incl;
        __syncthreads();
        uint32_t run = before + incl - mine;
        for (uint32_t w = 0; w < 1024u / 64u; ++w) {
          const uint32_t t = wave_total[w];
          run += w < wave ? t : 0u;
          before += t;
        }
#pragma unroll
        for (uint32_t j = 0; j < kPer; ++j) {
          if (at + j < mw) s.seen[at + j] = run;
          run += cnt[j];
        }
        __syncthreads();
      }
      // (at most K * cap / 2: each of them has two records at least)
      for (uint32_t i = threadIdx.x; i < before; i += blockDim.x) s.sums[i] = 0.f;
      __syncthreads();
      // a message names a coordinate at most once: no two threads add to the same sum
      for (uint32_t k = 0; k < a.K; ++k) {
        const uint32_t* const rp = s.pos(k);
        const uint32_t* const rv = s.val(k);
        const uint32_t n = s.count[k];
#pragma unroll 4
        for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
          const uint32_t p = rp[i], bits = s.multi[p >> 5], bit = 1u << (p & 31u);
          if (bits & bit) s.sums[s.seen[p >> 5] + (uint32_t)__popc(bits & (bit - 1u))] += __uint_as_float(rv[i]);
        }
        __syncthreads();   // message k is in before message k + 1 adds to the same coordinates
      }
      for (uint32_t w = threadIdx.x; w < mw; w += blockDim.x) {
        uint32_t bits = s.multi[w], at = bits ? s.seen[w] : 0u;
        for (; bits; bits &= bits - 1u, ++at) {
          const uint32_t p = w * 32u + (uint32_t)__ffs((int)bits) - 1u;
          x[p] = updated(a, x[p], s.sums[at]);
        }
      }
      return;
    }
    // (64 bits: a bucket may have 2^32 - 1 values, and the step past its end would come round)
    for (uint64_t p = threadIdx.x; p < m; p += blockDim.x) acc[p] = 0.f;
    __syncthreads();
    if (!open_strings(a, b, refs, &bad) || !parse_in_turns(a, refs, m, acc, &bad)) {
      if (threadIdx.x == 0) flag_corrupt(a.status);
      return;
    }
    for (uint64_t p = threadIdx.x; p < m; p += blockDim.x) x[p] = updated(a, x[p], acc[p]);
    return;
  }
  for (uint32_t e = threadIdx.x; e < L; e += blockDim.x) {
    lpos[e] = cl.pos[e]; lval[e] = cl.val[e]; lk[e] = (uint8_t)cl.msg[e];
  }
  __syncthreads();
  // entries of one coordinate hang on one chain
  for (uint32_t e = threadIdx.x; e < L; e += blockDim.x)
    next[e] = atomicExch(&head[(lpos[e] * 0x9E3779B9u) >> (32 - kHashBits)], e);
  __syncthreads();
  // (a message names a coordinate at most once: the terms of p are found in message order
  // by looking for the lowest message above the last one, terms + 1 walks along the chain)
  for (uint32_t e = threadIdx.x; e < L; e += blockDim.x) {
    const uint32_t p = lpos[e];
    const uint32_t first = head[(p * 0x9E3779B9u) >> (32 - kHashBits)];
    float sum = 0.f;
    int last = -1;
    for (;;) {
      uint32_t best = 0xFFFFFFFFu;
      float bestv = 0.f;
      for (uint32_t j = first; j != 0xFFFFFFFFu; j = next[j]) {
        const uint32_t kj = lk[j];
        if (lpos[j] == p && (int)kj > last && kj < best) { best = kj; bestv = lval[j]; }
      }
      if (best == 0xFFFFFFFFu) break;
      if (last < 0 && best != lk[e]) break;   // another thread holds the lowest message: its job
      sum += bestv;
      last = (int)best;
    }
    if (last >= 0) x[p] = updated(a, x[p], sum);
  }
}

// What adding a sum of +0 does to the coordinates that no message names: -0 becomes +0.
__global__ __launch_bounds__(256) void k_plus_zero(DecodeArgs a) {
  if (*a.status != 0) return;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < a.n; i += (uint64_t)gridDim.x * 256)
    if (__float_as_uint(a.x[i]) == 0x80000000u) a.x[i] = 0.f;
}

__global__ __launch_bounds__(256) void k_gen_apply(DecodeArgs a, const float* acc) {
  if (*a.status != 0) return;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < a.n; i += (uint64_t)gridDim.x * 256)
    a.x[i] = a.step ? fmaf(-a.c, acc[i], a.x[i]) : a.x[i] + acc[i];
}

// Fixed width, any bucket size: a thread has consecutive values of a bucket, eight of up to four bits and
// four wider ones, and takes the messages one after the other.  (The words of four messages
// requested together, eight values of any width: 28 thousand values, 16 bits, K = 14 19.0 us and 14.9 this way, as
// with a value per thread; 10M of d = 443, 8 bits, K = 4 35.9 and 31.2; 20M in one bucket, 8 bits, K = 4 56.0
// and 51.1, with a value per thread and 64-bit divisions 145; 20M of d = 60 thousand, 4 bits, K = 16 133 and 120.)
__host__ __device__ constexpr int fixed_values(int bits) { return bits <= 4 ? 8 : 4; }
template <int B>
__global__ __launch_bounds__(256) void k_gen_decode_fixed(DecodeArgs a) {
  if (*a.status != 0) return;
  constexpr uint32_t fmask = (1u << B) - 1u;
  constexpr int V = fixed_values(B), LW = V * B < 32 ? 1 : V * B / 32;   // level words of a thread's values
  const float s_f = (float)a.s;
  const uint32_t gpb = a.d / V + (a.d % V ? 1u : 0u);   // threads for a bucket
  const uint64_t total = (uint64_t)a.nb * gpb;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (uint64_t)gridDim.x * 256) {
    const uint64_t b = total >> 32 ? i / gpb : (uint32_t)i / gpb;
    const uint32_t e = (uint32_t)(i - b * gpb) * V;
    const uint64_t base = b * (uint64_t)a.d;
    const uint64_t m = min((uint64_t)a.d, a.n - base);
    if (e >= m) continue;
    const uint32_t here = (uint32_t)min(m - e, (uint64_t)V);
    const uint64_t lw = (m * B + 31) >> 5, sw = (m + 31) >> 5;
    const uint64_t off = (uint64_t)H_WORDS + b * (uint64_t)a.fixed_words_full;
    const uint64_t wi = ((uint64_t)e * B) >> 5;
    float* const x = a.x + base + e;
    float xv[V], sum[V];
    if (here == V) {
#pragma unroll
      for (int j = 0; j < V; j += 4) {
        const v4f_any p = *reinterpret_cast<const v4f_any*>(x + j);
        xv[j] = p.x; xv[j + 1] = p.y; xv[j + 2] = p.z; xv[j + 3] = p.w;
      }
    } else {
#pragma unroll
      for (uint32_t j = 0; j < V; ++j) xv[j] = j < here ? x[j] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < V; ++j) sum[j] = 0.f;
    for (uint32_t k = 0; k < a.K; ++k) {
      if (off + 2 + lw + sw > a.msg_words[k]) { flag_corrupt(a.status); continue; }
      const uint32_t* const str = a.msgs[k] + off;
      uint32_t lev[LW];
      if (wi + LW <= lw) {
#pragma unroll
        for (int w = 0; w < LW; ++w) lev[w] = str[2 + wi + w];
      } else {
#pragma unroll
        for (int w = 0; w < LW; ++w) lev[w] = wi + w < lw ? str[2 + wi + w] : 0u;
      }
      const uint32_t sign = str[2 + lw + (e >> 5)] >> (e & 31u);
      const float sc = __uint_as_float(str[0]) / s_f;
      const uint32_t esc = str[1] - e;              // (below V: one of these values)
      if (V * B < 32) lev[0] >>= (e * B) & 31u;
#pragma unroll
      for (uint32_t j = 0; j < V; ++j) {
        uint32_t z = (lev[j * B / 32] >> (j * B % 32)) & fmask;
        z = esc == j ? a.s : z;
        if (z > a.s && j < here) { flag_corrupt(a.status); z = 0; }
        const float mag = sc * (float)z;
        sum[j] += z && ((sign >> j) & 1u) ? -mag : mag;
      }
    }
#pragma unroll
    for (int j = 0; j < V; ++j) xv[j] = a.step ? fmaf(-a.c, sum[j], xv[j]) : xv[j] + sum[j];
    if (here == V) {
#pragma unroll
      for (int j = 0; j < V; j += 4) {
        v4f_any p;
        p.x = xv[j]; p.y = xv[j + 1]; p.z = xv[j + 2]; p.w = xv[j + 3];
        *reinterpret_cast<v4f_any*>(x + j) = p;
      }
    } else {
#pragma unroll
      for (uint32_t j = 0; j < V; ++j) if (j < here) x[j] = xv[j];
    }
  }
}

// ---- launchers -------------------------------------------------------------------------

hipError_t launch_gen_scale(const GenArgs& a, hipStream_t st) {
  const uint64_t per = kPartialWaves / group_size(a.spb), groups = a.nb * groups_of(a.spb);
  hipLaunchKernelGGL(k_gen_partial, dim3((uint32_t)((groups + per - 1) / per)), dim3(64 * kPartialWaves), 0, st, a);
  if (groups > a.nb) hipLaunchKernelGGL(k_gen_scale, dim3((uint32_t)a.nb), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_gen_encode(const GenArgs& a, bool aligned, hipStream_t st) {
  const dim3 grid((uint32_t)a.nseg), block(64);
  const size_t lds = 4 * ((size_t)a.sub_words + kRingWords);
#define QSGD_GEN(CODE)                                                                       \
  if (aligned) hipLaunchKernelGGL((k_gen_encode<CODE, true>), grid, block, lds, st, a);      \
  else hipLaunchKernelGGL((k_gen_encode<CODE, false>), grid, block, lds, st, a)
  if (a.code == QSGD_CODE_SPARSE) { QSGD_GEN(QSGD_CODE_SPARSE); }
  else if (a.code == QSGD_CODE_DENSE) { QSGD_GEN(QSGD_CODE_DENSE); }
  else { QSGD_GEN(QSGD_CODE_FIXED); }
#undef QSGD_GEN
  return hipGetLastError();
}
hipError_t launch_gen_scan(const GenArgs& a, uint32_t cus, hipStream_t st) {
  const uint32_t threads = a.spb <= 64 * kScanPer ? 64 : a.spb <= 256 * kScanPer ? 256 : 1024;
  hipLaunchKernelGGL(k_gen_scan, dim3((uint32_t)a.nb), dim3(threads), 0, st, a);
  if (a.nb > 1) {
    const uint32_t per = (uint32_t)((a.nb + cus - 1) / cus);
    hipLaunchKernelGGL(k_gen_table, dim3((uint32_t)((a.nb + per - 1) / per)), dim3(256), 0, st, a, per);
  }
  return hipGetLastError();
}
hipError_t launch_gen_place(const GenArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_gen_place, dim3((uint32_t)((a.nseg + 3) / 4)), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_gen_zero(float* p, uint64_t n, uint32_t blocks, hipStream_t st) {
  hipLaunchKernelGGL(k_gen_zero, dim3(blocks), dim3(256), 0, st, p, n);
  return hipGetLastError();
}
hipError_t launch_gen_parse(const DecodeArgs& a, float* acc, bool entries, hipStream_t st) {
  if (entries) {
    hipLaunchKernelGGL(k_gen_parse_entries, dim3(a.nb), dim3(256), 0, st, a, acc);
  } else {
    hipLaunchKernelGGL(k_gen_parse, dim3((a.nb + 255) / 256), dim3(256), 0, st, a, acc);
  }
  return hipGetLastError();
}
// area: n words; lists: a.nb x kCollideBytes behind it; stretches: about how many a string has; chunks:
// workgroups per list in `apply`.
hipError_t launch_sparse_long(const DecodeArgs& a, uint32_t* area, uint8_t* lists, uint32_t cus,
                              uint32_t stretches, uint32_t chunks, hipStream_t st) {
  const uint64_t clear = (uint64_t)a.nb * (2u * bitmap_words(a.d) + a.K);
  const uint64_t most = (uint64_t)cus * 32;
  const uint32_t blocks = (uint32_t)((clear + 255) / 256 < most ? (clear + 255) / 256 : most);
  hipLaunchKernelGGL(k_sparse_clear, dim3(blocks), dim3(256), 0, st, a, area, lists);
  hipLaunchKernelGGL(k_sparse_list, dim3(a.nb, a.K, stretches), dim3(kListThreads), 0, st, a, area, lists);
  if (!a.step || std::signbit(a.c))
    hipLaunchKernelGGL(k_plus_zero, dim3(cus * 32), dim3(256), 0, st, a);
  hipLaunchKernelGGL(k_sparse_apply, dim3(a.nb, a.K, chunks), dim3(256), 0, st, a, area, lists);
  hipLaunchKernelGGL(k_sparse_resolve, dim3(a.nb), dim3(1024), 0, st, a, area, lists);
  return hipGetLastError();
}
hipError_t launch_gen_apply(const DecodeArgs& a, const float* acc, uint32_t blocks, hipStream_t st) {
  hipLaunchKernelGGL(k_gen_apply, dim3(blocks), dim3(256), 0, st, a, acc);
  return hipGetLastError();
}
hipError_t launch_gen_decode_fixed(const DecodeArgs& a, uint32_t cus, hipStream_t st) {
  const uint32_t V = fixed_values((int)a.fixed_bits);
  const uint64_t threads = (uint64_t)a.nb * (a.d / V + (a.d % V ? 1u : 0u)), most = (uint64_t)cus * 1024;
  const dim3 grid((uint32_t)((threads + 255) / 256 < most ? (threads + 255) / 256 : most)), block(256);
  switch (a.fixed_bits) {
    case 2: hipLaunchKernelGGL(k_gen_decode_fixed<2>, grid, block, 0, st, a); break;
    case 4: hipLaunchKernelGGL(k_gen_decode_fixed<4>, grid, block, 0, st, a); break;
    case 8: hipLaunchKernelGGL(k_gen_decode_fixed<8>, grid, block, 0, st, a); break;
    default: hipLaunchKernelGGL(k_gen_decode_fixed<16>, grid, block, 0, st, a); break;
  }
  return hipGetLastError();
}

}  // namespace qsgd
