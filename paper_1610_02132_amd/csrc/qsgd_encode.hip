// Encode kernels: M <- Code(Q_s(g))  (Alg. 1; Q_s: Sec. 3.1 Eq. 2 per bucket of
// Sec. 4; Code_s / Code'_s: Sec. 3.1 and App. A.2-A.3; fixed-width: Sec. 5).
//
// Bucket path (d <= 8192, d % 4 == 0).  A team of TW wavefronts (= one
// workgroup) owns a contiguous run of buckets.  Per bucket: one coalesced
// float4 read of the data into registers, the scale by a wavefront shuffle
// reduction (fp64 accumulation), one Philox block per float4, stochastic
// rounding, code lengths, a wavefront prefix sum for bit offsets, and the code
// words OR-ed into an LDS image of the bucket's string.  Strings have
// data-dependent lengths, so a team appends them to its own region of the
// workspace and a second, small kernel moves the regions to their final place
// (exclusive sum over at most a few thousand team totals): no team ever waits
// for another one.  Fixed-width strings have closed-form offsets and go straight
// to the message.
#include <type_traits>

#include "qsgd_device.hpp"
#include "qsgd_encode_wave.hpp"
#include "qsgd_kernels.hpp"

#ifndef QSGD_UHI
#define QSGD_UHI 1
#endif
namespace qsgd {

namespace {

// Loads the float4 of this lane for the chunk starting `eoff` elements into the
// bucket; elements at or past m read as 0.
__device__ __forceinline__ float4 load_quad(const float* __restrict__ gb, uint32_t eoff,
                                            uint32_t m) {
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (eoff + 3 < m) {
    v = load_stream(gb + eoff);  // read once: the team's staged strings stay cached
  } else {
    if (eoff + 0 < m) v.x = gb[eoff + 0];
    if (eoff + 1 < m) v.y = gb[eoff + 1];
    if (eoff + 2 < m) v.z = gb[eoff + 2];
  }
  return v;
}

}  // namespace

// TW wavefronts per bucket, each holding up to CPW chunks of 256 elements.
// LIST (Code_s only): 0 = survivors go through a ring that is coded as it fills
// (encode_sparse_wave); list_records(CPW) = sparse data, survivors of all chunks are listed first
// (encode_sparse_list).
template <int TW, int CPW, int CODE, uint32_t LIST = 0>
__global__ __launch_bounds__(64 * TW)
    __attribute__((amdgpu_waves_per_eu(CODE == 2 ? 1 : (LIST ? QSGD_ENC_WAVES_LIST : QSGD_ENC_WAVES))))
    void k_encode_bucket(EncodeArgs a) {
  extern __shared__ uint32_t smem[];
  // LDS: [dst image of the bucket string][TW sub-streams][TW record rings][scratch]
  constexpr uint32_t kRingW = (CODE == QSGD_CODE_SPARSE) ? ring_words(LIST ? LIST : kRing) : 0u;
  uint32_t* const dst = smem;
  uint32_t* const sub_all = smem + a.dst_words;
  uint32_t* const ring_all = sub_all + TW * a.sub_words;
  double* const red = reinterpret_cast<double*>(ring_all + TW * kRingW);
  WaveOut* const winfo = reinterpret_cast<WaveOut*>(red + TW);
  uint32_t* const otab = reinterpret_cast<uint32_t*>(winfo + TW);  // kOmegaTab words (Code_s)

  const int tid = threadIdx.x;
  // (the wavefront's number is the same in all its lanes: as a scalar, what depends on it --
  // chunk bounds, LDS bases, the loop over chunks -- stays off the vector unit)
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  uint32_t* const sub = sub_all + wave * a.sub_words;
  uint32_t* const ring = ring_all + wave * kRingW;

  for (uint32_t j = tid; j < a.dst_words + TW * a.sub_words; j += 64 * TW) smem[j] = 0;
  if (CODE == QSGD_CODE_SPARSE) {
    for (uint32_t k = tid; k < kOmegaTab; k += 64 * TW) {
      uint64_t code = 0; uint32_t len = 0;
      if (k) omega_encode(k, code, len);
      otab[k] = ((uint32_t)code << 8) | len;
    }
  }

  if (blockIdx.x == 0 && tid == 0) {  // header; length and status are completed later
    uint32_t* h = a.header;
    h[H_MAGIC] = kMagic; h[H_VERSION] = a.version; h[H_CODE] = CODE; h[H_NORM] = a.norm_mode;
    h[H_S] = a.s; h[H_STREAM] = a.stream_id;
    h[H_D_LO] = (uint32_t)a.d; h[H_D_HI] = 0;
    h[H_N_LO] = (uint32_t)a.n; h[H_N_HI] = (uint32_t)(a.n >> 32);
    h[H_NB_LO] = a.nb; h[H_NB_HI] = 0;
    h[H_PW_LO] = (uint32_t)a.fixed_payload_words;
    h[H_PW_HI] = (uint32_t)(a.fixed_payload_words >> 32);
    h[H_STATUS] = 0; h[H_ITER] = a.iteration;
  }
  __syncthreads();

  const uint32_t b_begin = blockIdx.x * a.bper;
  const uint32_t b_end = min(b_begin + a.bper, a.nb);
  uint32_t* const region = a.staging + (uint64_t)blockIdx.x * a.region_words;
  uint32_t run = 0;  // words this team has appended to its region

  const uint32_t s = a.s;
  const float s_f = (float)s;

  // Extent of bucket b, as scalars: the same in every lane, and saying so keeps the bounds
  // and the addresses on the scalar unit.
  auto extent = [&](uint32_t b, uint64_t& base, uint32_t& m) {
    bucket_extent(a, b, base, m);
    base = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(base >> 32)) << 32) |
           __builtin_amdgcn_readfirstlane((uint32_t)base);
    m = __builtin_amdgcn_readfirstlane(m);
  };
  constexpr uint32_t kFull = (uint32_t)(TW * CPW) * kChunk;

  for (uint32_t b = b_begin; b < b_end; ++b) {
    uint64_t base;
    uint32_t m;
    extent(b, base, m);
    const float* __restrict__ gb = a.g + base;

    // ---- read the bucket once, accumulate the scale --------------------------
    float4 v[CPW];
    float mx = 0.f;
    if (m == kFull) {  // a full bucket: no bounds to check
#pragma unroll
      for (int c = 0; c < CPW; ++c)
        v[c] = load_stream(gb + (uint32_t)(wave * CPW + c) * kChunk + lane * 4);
    } else {
#pragma unroll
      for (int c = 0; c < CPW; ++c) {
        const uint32_t cstart = (uint32_t)(wave * CPW + c) * kChunk;
        v[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (cstart < m) v[c] = load_quad(gb, cstart + lane * 4, m);
      }
    }
    // the draws need no data: they are computed while the loads are in flight
    const uint32_t wstart = (uint32_t)wave * CPW * kChunk;  // bucket position of this wave
    QuantCtx qc;
    qc.inv = 0.f; qc.s_f = s_f; qc.s = s; qc.key0 = a.key0; qc.key1 = a.key1;
    qc.stream_id = a.stream_id; qc.iteration = a.iteration;
    uint32_t rall[CPW][4];
    draw_all<CPW, true>(a.index_base + base + wstart, lane, qc, rall);
    // squares are exact in fp64, so the fused multiply-add rounds like multiply, add
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
      if (a.norm_mode == 0) {
        s0 = fma((double)v[c].x, (double)v[c].x, s0);
        s1 = fma((double)v[c].y, (double)v[c].y, s1);
        s2 = fma((double)v[c].z, (double)v[c].z, s2);
        s3 = fma((double)v[c].w, (double)v[c].w, s3);
      } else {
        mx = fmaxf(fmaxf(mx, fmaxf(fabsf(v[c].x), fabsf(v[c].y))),
                   fmaxf(fabsf(v[c].z), fabsf(v[c].w)));
      }
    }
    double ss = (s0 + s1) + (s2 + s3);
    float scale;
    if (a.norm_mode == 0) {
      ss = wave_sum_f64(ss);
      if (TW > 1) {
        if (lane == 0) red[wave] = ss;
        __syncthreads();
        ss = 0.0;
#pragma unroll
        for (int w = 0; w < TW; ++w) ss += red[w];
      }
      scale = (float)sqrt(ss);
    } else {
      mx = wave_max_f32(mx);
      if (TW > 1) {
        if (lane == 0) red[wave] = (double)mx;
        __syncthreads();
        mx = 0.f;
#pragma unroll
        for (int w = 0; w < TW; ++w) mx = fmaxf(mx, (float)red[w]);
      }
      scale = mx;
    }
    const float inv = (scale > 0.f) ? s_f / scale : 0.f;

    // ---- fixed width: closed-form placement, straight to the message ---------
    if (CODE == QSGD_CODE_FIXED) {
      const uint32_t B = a.fixed_bits;
      const uint32_t fmax = (1u << B) - 1u;
      uint32_t* const str = a.payload + (uint64_t)b * a.fixed_words_full;
      const uint32_t lw = (m * B + 31u) >> 5, sw = (m + 31u) >> 5;
      uint32_t* const lplane = str + 2;
      uint32_t* const splane = lplane + lw;
      uint32_t esc = 0xFFFFFFFFu;
#pragma unroll
      for (int c = 0; c < CPW; ++c) {
        const uint32_t cstart = (uint32_t)(wave * CPW + c) * kChunk;
        if (cstart >= m) continue;
        const uint32_t e0 = cstart + lane * 4;
        const uint32_t (&r)[4] = rall[c];
        uint32_t z[4];
        z[0] = quantize_one(v[c].x, inv, s_f, s, r[0]);
        z[1] = quantize_one(v[c].y, inv, s_f, s, r[1]);
        z[2] = quantize_one(v[c].z, inv, s_f, s, r[2]);
        z[3] = quantize_one(v[c].w, inv, s_f, s, r[3]);
        const uint32_t nib = (v[c].x < 0.f ? 1u : 0u) | (v[c].y < 0.f ? 2u : 0u) |
                             (v[c].z < 0.f ? 4u : 0u) | (v[c].w < 0.f ? 8u : 0u);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (z[j] > fmax) { esc = e0 + j; z[j] = fmax; }
        // level plane: element i's field at bit i*B (LSB first)
        if (B == 8) {
          const uint32_t w = z[0] | (z[1] << 8) | (z[2] << 16) | (z[3] << 24);
          const uint32_t wi = e0 >> 2;
          if (wi < lw) lplane[wi] = w;
        } else if (B == 16) {
          const uint32_t wi = e0 >> 1;
          if (wi < lw) lplane[wi] = z[0] | (z[1] << 16);
          if (wi + 1 < lw) lplane[wi + 1] = z[2] | (z[3] << 16);
        } else if (B == 4) {
          uint32_t h = z[0] | (z[1] << 4) | (z[2] << 8) | (z[3] << 12);
          h |= dpp_fetch<kDppShl1, 0xf>(h) << 16;
          const uint32_t wi = e0 >> 3;
          if ((lane & 1) == 0 && wi < lw) lplane[wi] = h;
        } else {  // B == 2
          uint32_t h = z[0] | (z[1] << 2) | (z[2] << 4) | (z[3] << 6);
          h |= dpp_fetch<kDppShl1, 0xf>(h) << 8;
          h |= dpp_fetch<kDppShl2, 0xf>(h) << 16;
          const uint32_t wi = e0 >> 4;
          if ((lane & 3) == 0 && wi < lw) lplane[wi] = h;
        }
        // sign plane: element i at bit i%32 of word i/32
        uint32_t sg = nib;
        sg |= dpp_fetch<kDppShl1, 0xf>(sg) << 4;
        sg |= dpp_fetch<kDppShl2, 0xf>(sg) << 8;
        sg |= dpp_fetch<kDppShl4, 0xf>(sg) << 16;
        const uint32_t si = e0 >> 5;
        if ((lane & 7) == 0 && si < sw) splane[si] = sg;
      }
      // a short bucket inside a tensor-aware message keeps a full-size slot: zero its tail
      if (a.btab && m < a.d) {
        for (uint32_t w = 2u + lw + sw + (uint32_t)tid; w < a.fixed_words_full; w += 64 * TW)
          str[w] = 0;
      }
      // escape word: at most one lane of the team holds an index
      const uint64_t eb = __ballot(esc != 0xFFFFFFFFu);
      if (TW == 1) {
        if (eb) esc = lane_bcast(esc, __ffsll((unsigned long long)eb) - 1);
        if (lane == 0) { str[0] = __float_as_uint(scale); str[1] = esc; }
      } else {
        if (tid == 0) winfo[0].first_pos = 0xFFFFFFFFu;
        __syncthreads();
        if (esc != 0xFFFFFFFFu) winfo[0].first_pos = esc;
        __syncthreads();
        if (tid == 0) { str[0] = __float_as_uint(scale); str[1] = winfo[0].first_pos; }
        __syncthreads();
      }
      continue;
    }

    // ---- Elias codes: each wave builds its sub-stream in LDS -----------------
    qc.inv = inv;
    WaveOut wo;
    wo.first_pos = 0; wo.last_pos = 0; wo.bits = 0;
    {
      const uint32_t wlen = wstart < m ? min((uint32_t)CPW * kChunk, m - wstart) : 0u;
      const int nchunks = (int)((wlen + kChunk - 1) / kChunk);
      if (CODE == QSGD_CODE_SPARSE) {
        bool gave_up = false;
        if constexpr (LIST != 0) {
          gave_up = encode_sparse_list<CPW, LIST>(v, rall, nchunks, wstart, lane, qc, ring, otab,
                                                  sub, wo);
        } else {
          (void)encode_sparse_wave<CPW, false>(v, rall, nchunks, wstart, lane, qc, ring, otab, sub,
                                               wo);
        }
        if (LIST && gave_up) {
          // dense data after all: clear what the sub-stream holds and code the wavefront's
          // values chunk by chunk straight from memory
          const uint32_t dirty = min(a.sub_words, ((wo.bits + 31u) >> 5) + 2u);
          for (uint32_t j = lane; j < dirty; j += kWave) sub[j] = 0;
          wo.first_pos = 0; wo.last_pos = 0; wo.bits = 0;
          __builtin_amdgcn_wave_barrier();
#pragma unroll 1
          for (int c = 0; c < nchunks; ++c) {
            const uint32_t e0 = wstart + (uint32_t)c * kChunk + (uint32_t)lane * 4u;
            const float4 vc = load_quad(gb, e0, m);
            uint32_t rc[4];
            draw4<true>(a.index_base + base + e0, qc, rc);
            encode_sparse_direct<false>(vc, rc, e0 + 1u, lane, qc, sub, wo);
          }
        }
      } else {
        encode_dense_wave<CPW>(v, rall, nchunks, wlen, lane, qc, sub, wo);
      }
    }
    const uint32_t wbits = wo.bits;

    // ---- join the sub-streams into the bucket string --------------------------
    if (lane == 0) winfo[wave] = wo;
    __syncthreads();
    uint32_t cursor = 32;  // after the scale
    uint32_t my_start = 0, my_glen = 0, my_gap = 0;
    {
      uint32_t prev_last = 0;
#pragma unroll
      for (int w = 0; w < TW; ++w) {
        WaveOut wi;
        wi.first_pos = __builtin_amdgcn_readfirstlane(winfo[w].first_pos);
        wi.last_pos = __builtin_amdgcn_readfirstlane(winfo[w].last_pos);
        wi.bits = __builtin_amdgcn_readfirstlane(winfo[w].bits);
        uint32_t glen = 0, gap = 0;
        if (CODE == QSGD_CODE_SPARSE && wi.first_pos) {
          gap = wi.first_pos - prev_last;
          glen = omega_length(gap);
          prev_last = wi.last_pos;
        }
        if (w == wave) { my_start = cursor; my_glen = glen; my_gap = gap; }
        cursor += glen + wi.bits;
      }
    }
    const uint32_t stop = (CODE == QSGD_CODE_SPARSE) ? 1u : 0u;
    const uint32_t words = (cursor + stop + 31u) >> 5;
    if (tid == 0) {
      dst[0] = __float_as_uint(scale);
      if (stop) lds_emit(dst, cursor, 1ull, 1u);
    }
    if (lane == 0 && my_glen) {
      uint64_t gc; uint32_t gl;
      omega_encode(my_gap, gc, gl);
      lds_emit(dst, my_start, gc, gl);
    }
    {
      const uint32_t o = my_start + my_glen;
      const uint32_t w0 = o >> 5, sh = o & 31u;
      const uint32_t nsub = (wbits + 31u) >> 5;
      for (uint32_t j = lane; j < nsub; j += kWave) {
        const uint32_t x = sub[j];
        sub[j] = 0;
        if (x) {
          atomicOr(&dst[w0 + j], x >> sh);
          if (sh) atomicOr(&dst[w0 + j + 1], x << (32u - sh));
        }
      }
    }
    __syncthreads();

    // ---- append the string to the team's region --------------------------------
    // (a region smaller than the worst case may run out: the string is then dropped, the
    // count goes on, and the message ends up with the capacity status and the size needed)
    if (tid == 0) a.table[b] = run;  // relative to the region; rebased later
    const bool room = (uint64_t)run + words <= a.region_words;
    for (uint32_t j = tid; j < words; j += 64 * TW) {
      if (room) region[run + j] = dst[j];
      dst[j] = 0;
    }
    run += words;
    // no barrier here: the image is next written after two barriers of the next bucket
    // (scale exchange, sub-stream summaries), which every thread reaches after its zeroing
  }
  if (CODE != QSGD_CODE_FIXED && tid == 0) a.totals[blockIdx.x] = run;
}

// Fixed width, buckets of at most 1024 values: LPB lanes per bucket (64 / LPB buckets
// per wavefront at once), CP float4 per lane, B-bit fields.  Offsets are closed
// form, so the wavefront reads its buckets once and writes their strings in place;
// the per-bucket work (scale reduction, square root, divide) is shared by the
// buckets that ride in one wavefront.
template <int LPB, int CP, int B, bool ODD>
__device__ __forceinline__ void encode_fixed_small(const EncodeArgs& a) {
  constexpr int NB = 64 / LPB;             // buckets per wavefront pass
  constexpr uint32_t kStep = LPB * 4;      // values one pass of the bucket's lanes covers
  constexpr uint32_t fmax = (1u << B) - 1u;
  const int lane = threadIdx.x;
  const uint32_t sb = lane / LPB, l = lane % LPB;
  const int last_lane = (int)(sb * LPB + LPB - 1);

  if (blockIdx.x == 0 && lane == 0) {
    uint32_t* h = a.header;
    h[H_MAGIC] = kMagic; h[H_VERSION] = a.version; h[H_CODE] = QSGD_CODE_FIXED; h[H_NORM] = a.norm_mode;
    h[H_S] = a.s; h[H_STREAM] = a.stream_id;
    h[H_D_LO] = (uint32_t)a.d; h[H_D_HI] = 0;
    h[H_N_LO] = (uint32_t)a.n; h[H_N_HI] = (uint32_t)(a.n >> 32);
    h[H_NB_LO] = a.nb; h[H_NB_HI] = 0;
    h[H_PW_LO] = (uint32_t)a.fixed_payload_words;
    h[H_PW_HI] = (uint32_t)(a.fixed_payload_words >> 32);
    h[H_STATUS] = 0; h[H_ITER] = a.iteration;
  }
  const uint32_t s = a.s;
  const float s_f = (float)s;
  QuantCtx qc;
  qc.inv = 0.f; qc.s_f = s_f; qc.s = s; qc.key0 = a.key0; qc.key1 = a.key1;
  qc.stream_id = a.stream_id; qc.iteration = a.iteration;

  const uint32_t g_begin = blockIdx.x * a.bper;               // bucket groups of this team
  const uint32_t g_end = min(g_begin + a.bper, (a.nb + NB - 1) / NB);
  for (uint32_t grp = g_begin; grp < g_end; ++grp) {
    const uint32_t b = grp * NB + sb;
    const bool live = b < a.nb;
    uint64_t base = 0;
    uint32_t m = 0;
    if (live) bucket_extent(a, b, base, m);
    const float* __restrict__ gb = a.g + base;
    // every lane's CP quads lie inside its bucket: no per-element bounds needed
    const bool all_full = __ballot(m == (uint32_t)CP * kStep) == ~0ull;

    float4 v[CP];
    uint32_t r[CP][4];
#pragma unroll
    for (int c = 0; c < CP; ++c) {
      const uint32_t e0 = (uint32_t)c * kStep + l * 4;
      auto quad = [&]() {
        if constexpr (ODD) {
          const v4f_any t = *reinterpret_cast<const v4f_any*>(gb + e0);
          return make_float4(t.x, t.y, t.z, t.w);
        } else {
          return *reinterpret_cast<const float4*>(gb + e0);
        }
      };
      if (all_full) {
        v[c] = quad();
      } else {
        v[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (e0 + 3 < m) {
          v[c] = quad();
        } else {
          if (e0 + 0 < m) v[c].x = gb[e0 + 0];
          if (e0 + 1 < m) v[c].y = gb[e0 + 1];
          if (e0 + 2 < m) v[c].z = gb[e0 + 2];
        }
      }
    }
    {
      const uint64_t g0 = a.index_base + base + l * 4;
      uint32_t hi;
      if constexpr (ODD) {
#pragma unroll
        for (int c = 0; c < CP; ++c) draw4<false>(g0 + (uint64_t)c * kStep, qc, r[c]);
      } else if (QSGD_UHI && uniform_counter_hi(g0, g0 + (uint64_t)(CP - 1) * kStep, hi)) {
#pragma unroll
        for (int c = 0; c < CP; ++c) draw4_uniform_hi(g0 + (uint64_t)c * kStep, hi, qc, r[c]);
      } else {
#pragma unroll
        for (int c = 0; c < CP; ++c) draw4<true>(g0 + (uint64_t)c * kStep, qc, r[c]);
      }
    }

    // ---- scale of each bucket: reduction over its LPB lanes -------------------------
    float scale;
    if (a.norm_mode == 0) {
      double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
      for (int c = 0; c < CP; ++c) {
        s0 = fma((double)v[c].x, (double)v[c].x, s0);
        s1 = fma((double)v[c].y, (double)v[c].y, s1);
        s2 = fma((double)v[c].z, (double)v[c].z, s2);
        s3 = fma((double)v[c].w, (double)v[c].w, s3);
      }
      double ss = (s0 + s1) + (s2 + s3);
      ss += dpp_fetch_f64<kDppShr1, 0xf>(ss);
      ss += dpp_fetch_f64<kDppShr2, 0xf>(ss);
      ss += dpp_fetch_f64<kDppShr4, 0xf>(ss);
      ss += dpp_fetch_f64<kDppShr8, 0xf>(ss);
      if (LPB >= 32) ss += dpp_fetch_f64<kDppBcast15, 0xa>(ss);
      if (LPB >= 64) ss += dpp_fetch_f64<kDppBcast31, 0xc>(ss);
      scale = (float)sqrt(ss);  // right in the last lane of each bucket
    } else {
      float mx = 0.f;
#pragma unroll
      for (int c = 0; c < CP; ++c)
        mx = fmaxf(fmaxf(mx, fmaxf(fabsf(v[c].x), fabsf(v[c].y))),
                   fmaxf(fabsf(v[c].z), fabsf(v[c].w)));
      mx = fmaxf(mx, __uint_as_float(dpp_fetch<kDppShr1, 0xf>(__float_as_uint(mx))));
      mx = fmaxf(mx, __uint_as_float(dpp_fetch<kDppShr2, 0xf>(__float_as_uint(mx))));
      mx = fmaxf(mx, __uint_as_float(dpp_fetch<kDppShr4, 0xf>(__float_as_uint(mx))));
      mx = fmaxf(mx, __uint_as_float(dpp_fetch<kDppShr8, 0xf>(__float_as_uint(mx))));
      if (LPB >= 32) mx = fmaxf(mx, __uint_as_float(dpp_fetch<kDppBcast15, 0xa>(__float_as_uint(mx))));
      if (LPB >= 64) mx = fmaxf(mx, __uint_as_float(dpp_fetch<kDppBcast31, 0xc>(__float_as_uint(mx))));
      scale = mx;
    }
    scale = __shfl(scale, last_lane, kWave);
    const float inv = (scale > 0.f) ? s_f / scale : 0.f;

    // ---- quantize, pack, store ------------------------------------------------------------
    uint32_t* const str = a.payload + (uint64_t)b * a.fixed_words_full;
    const uint32_t lw = (m * B + 31u) >> 5, sw = (m + 31u) >> 5;
    uint32_t* const lplane = str + 2;
    uint32_t* const splane = lplane + lw;
    uint32_t esc = 0xFFFFFFFFu;
    const uint32_t zlim = min(fmax, s);
#pragma unroll
    for (int c = 0; c < CP; ++c) {
      const uint32_t e0 = (uint32_t)c * kStep + l * 4;
      uint32_t z[4];
      z[0] = quantize_unclamped(v[c].x, inv, r[c][0]);
      z[1] = quantize_unclamped(v[c].y, inv, r[c][1]);
      z[2] = quantize_unclamped(v[c].z, inv, r[c][2]);
      z[3] = quantize_unclamped(v[c].w, inv, r[c][3]);
      const uint32_t nib = (v[c].x < 0.f ? 1u : 0u) | (v[c].y < 0.f ? 2u : 0u) |
                           (v[c].z < 0.f ? 4u : 0u) | (v[c].w < 0.f ? 8u : 0u);
      // rare: a level above s (clamped to s here) or one the field cannot hold (level s
      // with s = 2^B, which goes to the escape word)
      if (max(max(z[0], z[1]), max(z[2], z[3])) > zlim) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          z[j] = min(z[j], s);
          if (z[j] > fmax) { esc = e0 + j; z[j] = fmax; }
        }
      }
      if (B == 8) {
        const uint32_t wi = e0 >> 2;
        if (all_full || wi < lw) lplane[wi] = z[0] | (z[1] << 8) | (z[2] << 16) | (z[3] << 24);
      } else if (B == 16) {
        const uint32_t wi = e0 >> 1;
        if (all_full || wi < lw) lplane[wi] = z[0] | (z[1] << 16);
        if (all_full || wi + 1 < lw) lplane[wi + 1] = z[2] | (z[3] << 16);
      } else if (B == 4) {
        uint32_t h = z[0] | (z[1] << 4) | (z[2] << 8) | (z[3] << 12);
        h |= dpp_fetch<kDppShl1, 0xf>(h) << 16;
        const uint32_t wi = e0 >> 3;
        if ((l & 1) == 0 && (all_full || wi < lw)) lplane[wi] = h;
      } else {
        uint32_t h = z[0] | (z[1] << 2) | (z[2] << 4) | (z[3] << 6);
        h |= dpp_fetch<kDppShl1, 0xf>(h) << 8;
        h |= dpp_fetch<kDppShl2, 0xf>(h) << 16;
        const uint32_t wi = e0 >> 4;
        if ((l & 3) == 0 && (all_full || wi < lw)) lplane[wi] = h;
      }
      uint32_t sg = nib;
      sg |= dpp_fetch<kDppShl1, 0xf>(sg) << 4;
      sg |= dpp_fetch<kDppShl2, 0xf>(sg) << 8;
      sg |= dpp_fetch<kDppShl4, 0xf>(sg) << 16;
      const uint32_t si = e0 >> 5;
      if ((l & 7) == 0 && (all_full || si < sw)) splane[si] = sg;
    }
    // a short bucket inside a tensor-aware message keeps a full-size slot: zero its tail
    if (a.btab && live && m < a.d) {
      for (uint32_t w = 2u + lw + sw + l; w < a.fixed_words_full; w += LPB) str[w] = 0;
    }
    // escape word of each bucket: at most one of its lanes holds an index
    const uint64_t eb = __ballot(esc != 0xFFFFFFFFu);
    if (eb) {
      uint64_t mine = eb;
      if constexpr (LPB < 64) mine = (eb >> (sb * LPB)) & ((1ull << LPB) - 1ull);
      const int src = mine ? (int)(sb * LPB) + __ffsll((unsigned long long)mine) - 1 : lane;
      const uint32_t got = (uint32_t)__shfl((int)esc, src, kWave);
      esc = mine ? got : 0xFFFFFFFFu;
    }
    if (l == 0 && live) {
      str[0] = __float_as_uint(scale);
      str[1] = esc;
    }
  }
}

template <int LPB, int CP, int B, bool ODD>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(QSGD_FS_WAVES)))
void k_encode_fixed_small(EncodeArgs a) {
  encode_fixed_small<LPB, CP, B, ODD>(a);
}

// The K gradients of a double-buffered pass's chunk in one launch: a chunk of 16M values alone is
// 16 thousand wavefronts, four rounds of what the machine holds, and ran at 3.7 TB/s; eight of
// them together (4 bits, d = 512) take 113 us, 5.2 TB/s.
template <int LPB, int CP, int B>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(QSGD_FS_WAVES)))
void k_encode_fixed_small_batch(EncodeArgs a, EncodeBatch batch) {
  const uint32_t k = blockIdx.y;
  a.g = batch.g[k];
  a.header = batch.msg[k];
  a.payload = batch.msg[k] + H_WORDS;
  a.stream_id += k;
  encode_fixed_small<LPB, CP, B, false>(a);
}

// Moves each team's region to its place in the message: base_j = words of the teams
// before j.  A workgroup has `tpb` consecutive teams, a wavefront one of them at a time;
// it adds up the totals before its first team itself (at most kMaxTeams words, 16 bytes a
// load, from the L2) instead of reading prefix sums that a launch of its own would have to
// make first.  Bound by latency: with that launch and its gap 5.2 us at 40 teams and 15.4
// at 7143 (25.6M values), without it 2.6 and 9.8.
constexpr uint32_t kCompactWaves = 4;
typedef uint32_t v4u_any __attribute__((ext_vector_type(4), aligned(4)));
//
// AHEAD: a team's words are requested before its place is known, those of a wavefront's first team before the
// totals are added up, those of its next one when this one is stored (25.6M values, 7143 teams: 9.8 -> 7.2 us).
// Where a team has few words there is little to wait for and more to issue (20 thousand values: 3.36 and 3.68).
//
// RAW: the workgroups behind the teams' copy the small tensors of a tensor-aware message, a piece of
// kRawPiece values each, behind all strings.  (A launch of their own took 4.7 us.)
template <bool RAW, bool AHEAD>
__global__ __launch_bounds__(64 * kCompactWaves) void k_encode_compact(CompactArgs a, RawArgs r) {
  __shared__ unsigned long long part[kCompactWaves];
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane((uint32_t)tid >> 6);
  const uint32_t groups = (a.teams + a.tpb - 1) / a.tpb;
  const bool raw = RAW && blockIdx.x >= groups;
  const uint32_t t_begin = raw ? a.teams : blockIdx.x * a.tpb;
  const uint32_t t_end = min(t_begin + a.tpb, a.teams);

  // (tpb <= 64: lane l keeps the total of the workgroup's team l)
  const uint32_t own = t_begin + (uint32_t)lane < t_end ? a.totals[t_begin + lane] : 0u;
  // AHEAD: the wavefront's next team, in registers as far as it goes
  constexpr uint32_t kQuads = 4;
  uint4 next[kQuads];
  uint32_t next_off = 0;
  auto request = [&](uint32_t i) {   // team t_begin + i
    if (!AHEAD || t_begin + i >= t_end) return;
    const uint32_t mine = lane_bcast(own, (int)i), j = t_begin + i;
    if (mine <= a.region_words) {   // (regions start on 16 bytes and hold whole quads)
      const uint4* const src = reinterpret_cast<const uint4*>(a.staging + (uint64_t)j * a.region_words);
#pragma unroll
      for (uint32_t u = 0; u < kQuads; ++u)
        if (4u * (u * kWave + lane) < mine) next[u] = src[u * kWave + lane];
    }
    const uint32_t b = j * a.bper + lane;
    if (lane < (int)min(a.bper, (uint32_t)kWave) && b < a.nb) next_off = a.table[b];
  };
  request(wave);
  // words of the teams before this workgroup's first one
  unsigned long long sum = 0;
  const uint4* const q = reinterpret_cast<const uint4*>(a.totals);
  const uint32_t quads = t_begin >> 2;
#pragma unroll 4
  for (uint32_t i = tid; i < quads; i += 64 * kCompactWaves) {
    const uint4 v = q[i];
    sum += ((unsigned long long)v.x + v.y) + ((unsigned long long)v.z + v.w);
  }
  if ((uint32_t)tid < (t_begin & 3u)) sum += a.totals[4u * quads + tid];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, kWave);
  if (lane == 0) part[wave] = sum;
  __syncthreads();
  unsigned long long base = 0;
#pragma unroll
  for (uint32_t w = 0; w < kCompactWaves; ++w) base += part[w];

  if constexpr (RAW) {
    if (raw) {
      // (where a string did not fit the message is void, whatever stands in it)
      if (base + r.raw_words > a.cap_words) return;
      const uint4 e = r.rtab[blockIdx.x - groups];
      const float* __restrict__ src = r.g + (uint64_t)e.x * 4u;
      uint32_t* __restrict__ dst = a.payload + base + e.z;
      const uint32_t i = (uint32_t)tid * 4u;
      if (i + 3u < e.y) {
        const v4u_any v = *reinterpret_cast<const v4u_any*>(src + i);   // tensors start at 16-byte multiples
        *reinterpret_cast<v4u_any*>(dst + i) = v;
      } else {
        for (uint32_t j = i; j < e.y; ++j) dst[j] = __float_as_uint(src[j]);
      }
      return;
    }
  }

  bool all_fit = true;
  for (uint32_t j = t_begin; j < t_end; ++j) {
    const uint32_t mine = lane_bcast(own, (int)(j - t_begin));
    // (a team whose region ran out has counted on without storing: nothing to copy)
    const bool fits = base + mine <= a.cap_words && base + mine <= 0xFFFFFFFFull &&
                      mine <= a.region_words;
    all_fit = all_fit && fits;
    if ((j - t_begin) % kCompactWaves == wave) {
      if (fits) {
        const uint32_t* __restrict__ src = a.staging + (uint64_t)j * a.region_words;
        uint32_t* __restrict__ dstp = a.payload + base;
#pragma unroll
        for (uint32_t u = 0; u < (AHEAD ? kQuads : 0u); ++u) {
          const uint32_t i = 4u * (u * kWave + lane);
          if (i + 4u <= mine) {
            v4u_any x; x.x = next[u].x; x.y = next[u].y; x.z = next[u].z; x.w = next[u].w;
            *reinterpret_cast<v4u_any*>(dstp + i) = x;
          } else if (i < mine) {
            dstp[i] = next[u].x;
            if (i + 1u < mine) dstp[i + 1u] = next[u].y;
            if (i + 2u < mine) dstp[i + 2u] = next[u].z;
          }
        }
#pragma unroll 4
        for (uint32_t i = (AHEAD ? 4u * kQuads * kWave : 0u) + lane; i < mine; i += kWave) dstp[i] = src[i];
      }
      const uint32_t b_begin = j * a.bper;
      const uint32_t b_end = min(b_begin + a.bper, a.nb);
      if (AHEAD && b_begin + lane < b_end) a.table[b_begin + lane] = (uint32_t)min(base + next_off, 0xFFFFFFFFull);
      for (uint32_t b = b_begin + (AHEAD ? kWave : 0u) + lane; b < b_end; b += kWave)
        a.table[b] = (uint32_t)min(base + a.table[b], 0xFFFFFFFFull);
      request(j - t_begin + kCompactWaves);
    }
    base += mine;
  }
  if (tid == 0) {
    if (!all_fit) atomicExch(&a.header[H_STATUS], (uint32_t)QSGD_ERR_CAPACITY);
    if (t_end == a.teams) {
      a.table[a.nb] = (uint32_t)min(base, 0xFFFFFFFFull);
      for (uint32_t i = a.nb + 1; i < a.table_words; ++i) a.table[i] = 0;  // padding
      const uint64_t all = base + a.raw_words;   // the raw values follow the strings
      if (all > a.cap_words) atomicExch(&a.header[H_STATUS], (uint32_t)QSGD_ERR_CAPACITY);
      a.header[H_PW_LO] = (uint32_t)all;
      a.header[H_PW_HI] = (uint32_t)(all >> 32);
    }
  }
}

// Header of an empty message (n = 0).
__global__ void k_write_empty(uint32_t* header, uint32_t* table, uint32_t code, uint32_t norm,
                              uint32_t s, uint64_t d, uint32_t stream_id, uint32_t iteration) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    header[H_MAGIC] = kMagic; header[H_VERSION] = 1; header[H_CODE] = code;
    header[H_NORM] = norm; header[H_S] = s; header[H_STREAM] = stream_id;
    header[H_D_LO] = (uint32_t)d; header[H_D_HI] = (uint32_t)(d >> 32);
    header[H_N_LO] = 0; header[H_N_HI] = 0; header[H_NB_LO] = 0; header[H_NB_HI] = 0;
    header[H_PW_LO] = 0; header[H_PW_HI] = 0; header[H_STATUS] = 0;
    header[H_ITER] = iteration;
    if (table) { table[0] = 0; table[1] = 0; table[2] = 0; table[3] = 0; }
  }
}

// ---- launch table -------------------------------------------------------------
// (d <= 2048: Elias codes mostly take launch_encode_direct, fixed width up to 1024
// launch_encode_fixed_small)
template <int TW, int CPW, int CODE, uint32_t LIST = 0>
static hipError_t launch_bucket(const EncodeArgs& a, uint32_t teams, size_t lds, hipStream_t st) {
  hipLaunchKernelGGL((k_encode_bucket<TW, CPW, CODE, LIST>), dim3(teams), dim3(64 * TW), lds, st, a);
  return hipGetLastError();
}

template <int TW>
static hipError_t launch_team(const EncodeArgs& a, uint32_t code, uint32_t teams, size_t lds,
                              hipStream_t st) {
  switch (code) {
    case QSGD_CODE_SPARSE:
      return a.ring == list_records(8)
                 ? launch_bucket<TW, 8, QSGD_CODE_SPARSE, list_records(8)>(a, teams, lds, st)
                 : launch_bucket<TW, 8, QSGD_CODE_SPARSE>(a, teams, lds, st);
    case QSGD_CODE_DENSE: return launch_bucket<TW, 8, QSGD_CODE_DENSE>(a, teams, lds, st);
    default: return launch_bucket<TW, 8, QSGD_CODE_FIXED>(a, teams, lds, st);
  }
}

hipError_t launch_encode_bucket(const EncodeArgs& a, uint32_t code, int tw, int cpw,
                                uint32_t teams, size_t lds, hipStream_t st) {
  if (tw == 1 && cpw == 4 && code == QSGD_CODE_SPARSE)
    return launch_bucket<1, 4, QSGD_CODE_SPARSE>(a, teams, lds, st);
  if (tw == 1 && cpw == 8 && code == QSGD_CODE_FIXED)
    return launch_bucket<1, 8, QSGD_CODE_FIXED>(a, teams, lds, st);
  if (tw == 2 && cpw == 8) return launch_team<2>(a, code, teams, lds, st);
  if (tw == 4 && cpw == 8) return launch_team<4>(a, code, teams, lds, st);
  return hipErrorInvalidValue;
}

// f(lanes per bucket, float4 per lane, field bits), all as compile-time constants
template <class F>
static void fixed_small_shape(int lpb, int cp, uint32_t bits, F&& f) {
  auto field = [&](auto l, auto c) {
    switch (bits) {
      case 2: f(l, c, std::integral_constant<int, 2>()); break;
      case 4: f(l, c, std::integral_constant<int, 4>()); break;
      case 8: f(l, c, std::integral_constant<int, 8>()); break;
      default: f(l, c, std::integral_constant<int, 16>()); break;
    }
  };
  using std::integral_constant;
  if (lpb == 16 && cp <= 1) field(integral_constant<int, 16>(), integral_constant<int, 1>());
  else if (lpb == 16 && cp <= 2) field(integral_constant<int, 16>(), integral_constant<int, 2>());
  else if (lpb == 16) field(integral_constant<int, 16>(), integral_constant<int, 4>());
  else if (lpb == 32) field(integral_constant<int, 32>(), integral_constant<int, 4>());
  else field(integral_constant<int, 64>(), integral_constant<int, 4>());
}

// d <= 1024; a.bper counts groups of 64/lpb buckets per team.  (Bucket sizes off 4 take unaligned loads
// and two Philox blocks per quad; 10M values on the general path, a wavefront or more per bucket, and
// here: d = 443, s = 255 64 and 18 us, d = 41, s = 15 467 and 26.)
hipError_t launch_encode_fixed_small(const EncodeArgs& a, int lpb, int cp, uint32_t teams,
                                     hipStream_t st) {
  fixed_small_shape(lpb, cp, a.fixed_bits, [&](auto l, auto c, auto b) {
    constexpr int L = decltype(l)::value, C = decltype(c)::value, B = decltype(b)::value;
    if (a.d % 4) hipLaunchKernelGGL((k_encode_fixed_small<L, C, B, true>), dim3(teams), dim3(64), 0, st, a);
    else hipLaunchKernelGGL((k_encode_fixed_small<L, C, B, false>), dim3(teams), dim3(64), 0, st, a);
  });
  return hipGetLastError();
}

hipError_t launch_encode_fixed_small_batch(const EncodeArgs& a, const EncodeBatch& batch, uint32_t K,
                                           int lpb, int cp, uint32_t teams, hipStream_t st) {
  fixed_small_shape(lpb, cp, a.fixed_bits, [&](auto l, auto c, auto b) {
    hipLaunchKernelGGL((k_encode_fixed_small_batch<decltype(l)::value, decltype(c)::value, decltype(b)::value>),
                       dim3(teams, K), dim3(64), 0, st, a, batch);
  });
  return hipGetLastError();
}

static_assert(kRawPiece == 4 * 64 * kCompactWaves, "a piece per workgroup, four values per thread");
hipError_t launch_encode_compact(const CompactArgs& a, const RawArgs* raw, bool ahead, hipStream_t st) {
  const uint32_t groups = (a.teams + a.tpb - 1) / a.tpb;
  const dim3 block(64 * kCompactWaves);
  const bool with_raw = raw && raw->R;
  const RawArgs r = with_raw ? *raw : RawArgs();
  const dim3 grid(groups + (with_raw ? raw->R : 0));
  if (ahead) {
    if (with_raw) hipLaunchKernelGGL((k_encode_compact<true, true>), grid, block, 0, st, a, r);
    else hipLaunchKernelGGL((k_encode_compact<false, true>), grid, block, 0, st, a, r);
  } else {
    if (with_raw) hipLaunchKernelGGL((k_encode_compact<true, false>), grid, block, 0, st, a, r);
    else hipLaunchKernelGGL((k_encode_compact<false, false>), grid, block, 0, st, a, r);
  }
  return hipGetLastError();
}

hipError_t launch_write_empty(uint32_t* header, uint32_t* table, uint32_t code, uint32_t norm,
                              uint32_t s, uint64_t d, uint32_t stream_id, uint32_t iteration,
                              hipStream_t st) {
  hipLaunchKernelGGL(k_write_empty, dim3(1), dim3(64), 0, st, header, table, code, norm, s, d,
                     stream_id, iteration);
  return hipGetLastError();
}

}  // namespace qsgd
