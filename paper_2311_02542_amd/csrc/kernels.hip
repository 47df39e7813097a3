// Kernels of the renderer hot path and their launchers.
//
// render_kernel is the whole per-ray path in one launch (the paper's
// single-kernel interleave of ray marching, hash sampling and MLPs, Sec. 5):
// persistent waves own 64 rays each (one per lane); every round a wave
//   1. takes the rays of the next 8x8 pixel tile when its own have all ended,
//      from a per-XCD queue (XCD-aware: block b works the queue of XCD b % 8
//      first, whose tiles come in long runs, so each XCD's L2 sees coherent
//      regions);
//   2. marches every ray to its next occupied lattice sample (bounded
//      number of lattice tests per round, empty bricks skipped);
//   3. compacts the lanes that found a sample into 16-sample tiles and, per
//      tile, encodes the hash grid (4 lanes per sample, levels interleaved
//      so LOD-skipped fine levels idle all lane groups equally) and runs the
//      density and color MLPs on MFMA with the activations in registers;
//   4. composites in FP32 and retires rays at T < t_min, at the sample cap
//      or when the march leaves the grid, writing RGBA and sample counts.
// Counters in the workspace return to zero when the last block finishes, so
// the launch needs no memset and can be replayed from a HIP graph.
//
// A launch that does not fill the chip is bound by the latency of a wave's
// rounds, one 16-sample tile after the other.  Its waves carry 16 or 32 rays
// instead of 64 (RenderArgs::lanes), one or two tiles a round, and more waves
// share the rays.
#include <map>
#include <mutex>
#include <type_traits>

#include "device.hpp"

namespace vrn {

#ifdef VRN_DEBUG_CHECKS
__device__ unsigned long long vrn_debug_counts[kDbgSlots];
#endif

constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr uint32_t kHelped = 2;      // other queues a wave takes rays from when its own is empty

#ifdef VRN_PHASE_TIMING
__device__ unsigned long long vrn_phase_cycles[kPhaseSlots];
#define VRN_PHASE_START()                              \
  unsigned long long ph_[kPhaseSlots] = {};            \
  unsigned long long tph_ = __builtin_amdgcn_s_memtime()
#define VRN_PHASE(slot)                                               \
  do {                                                                \
    const unsigned long long tn_ = __builtin_amdgcn_s_memtime();     \
    ph_[(slot)] += tn_ - tph_;                                        \
    tph_ = tn_;                                                       \
  } while (0)
#define VRN_PHASE_FLUSH()                                                                  \
  do {                                                                                     \
    if (lane_id() == 0)                                                                    \
      for (int i_ = 0; i_ < kPhaseSlots; ++i_) atomicAdd(&vrn_phase_cycles[i_], ph_[i_]); \
  } while (0)
#else
#define VRN_PHASE_START() \
  do {                    \
  } while (0)
#define VRN_PHASE(slot) \
  do {                  \
  } while (0)
#define VRN_PHASE_FLUSH() \
  do {                    \
  } while (0)
#endif

// exp for compositing: the FP32 path keeps the library expf; the 16-bit
// paths, whose inputs carry FP16 rounding already, use the hardware
// exponential (one multiply and v_exp_f32).
template <bool FAST>
__device__ __forceinline__ float comp_exp(float z) {
  if constexpr (FAST) return __expf(z);
  else return expf(z);
}

template <bool FAST>
__device__ __forceinline__ float sigmoidf(float z) { return __builtin_amdgcn_rcpf(1.0f + comp_exp<FAST>(-z)); }

// MLP arithmetic of a compute mode: 0 FP32 MFMA, 1 FP16, 2 BF16, 3 FP32 by
// split BF16 (VRN_F32X).  Modes 0 and 3 share everything but the MLP: the
// FP32 encode, FP32 SH values and the library exp in compositing.
template <int MODE>
constexpr bool kF32Class = MODE == 0 || MODE == 3;

// Bytes of the split weights of mode 3 in LDS: three BF16 parts, then the
// FP32 fragments of the color output layer (run on the VALU).
constexpr int kX3Bytes = 3 * kW16Total * 2;

template <int MODE>
struct WeightSmem {
  static constexpr int kBytes =
      (MODE == 0) ? kW32Total * 4 : (MODE == 3 ? kX3Bytes + (kW32Total - kW32_C3) * 4 : kW16Total * 2);
};

template <int MODE>
__device__ __forceinline__ const uint4* weight_src(const FieldDev& F) {
  if constexpr (MODE == 0) return reinterpret_cast<const uint4*>(F.w32);
  else if constexpr (MODE == 1) return reinterpret_cast<const uint4*>(F.w16);
  else if constexpr (MODE == 2) return reinterpret_cast<const uint4*>(F.wbf);
  else return reinterpret_cast<const uint4*>(F.wx3);
}

// Copy n 16-byte words to LDS with a block of any size, eight loads a thread in
// flight: with one, the 20 to 70 of a small launch's one-wave blocks came one
// after the other (256^2 FP16 frame 76 -> 67 us, together with the end of
// launches whose rays are all dealt).
__device__ __forceinline__ void stage(uint4* dst, const uint4* __restrict__ src, uint32_t n) {
  for (uint32_t i = threadIdx.x; i < n; i += 8u * blockDim.x) {
    uint4 v[8];
#pragma unroll
    for (uint32_t k = 0; k < 8u; ++k) v[k] = src[min(i + k * blockDim.x, n - 1u)];
#pragma unroll
    for (uint32_t k = 0; k < 8u; ++k)
      if (i + k * blockDim.x < n) dst[i + k * blockDim.x] = v[k];
  }
}

template <int MODE>
__device__ __forceinline__ void load_weights(const FieldDev& F, uint8_t* s_w, float* s_b) {
  uint4* dst = reinterpret_cast<uint4*>(s_w);
  constexpr int kMain = MODE == 3 ? kX3Bytes : WeightSmem<MODE>::kBytes;
  stage(dst, weight_src<MODE>(F), kMain / 16);
  if constexpr (MODE == 3)
    stage(dst + kX3Bytes / 16, reinterpret_cast<const uint4*>(F.w32 + kW32_C3), (kW32Total - kW32_C3) / 4);
  for (int i = threadIdx.x; i < kBiasTotal; i += blockDim.x) s_b[i] = F.bias[i];
}

template <int MODE>
__device__ __forceinline__ void run_mlp(const uint8_t* s_w, const float* s_b, const FieldDev& F,
                                        const float feat[8], const float shs[4], int lane, float& o0,
                                        float lg[3]) {
  if constexpr (MODE == 0)
    mlp_tile_f32(reinterpret_cast<const float4*>(s_w), s_b, F.d1_ksteps / 4, feat, shs, lane, o0, lg);
  else if constexpr (MODE == 3)
    mlp_tile_x3(reinterpret_cast<const uint4*>(s_w), reinterpret_cast<const float4*>(s_w + kX3Bytes), s_b, feat,
                shs, lane, o0, lg);
  else {
    typedef Half8<MODE == 2> H;
    const typename H::vec xin[1] = {H::pack(feat)};
    const uint2 shh[1] = {H::pack4(shs)};
    float o[1], l[1][3];
    mlp_batch_16<MODE == 2, 1>(reinterpret_cast<const uint4*>(s_w), s_b, 1, xin, shh, lane, o, l);
    o0 = o[0];
    for (int c = 0; c < 3; ++c) lg[c] = l[0][c];
  }
}

// The lane that owns compacted sample s = 16 t + (lane & 15), from the
// wave's slot table in LDS.
__device__ __forceinline__ int tile_source(const uint32_t* s_slot_w, int ns, int t, int lane, bool& act) {
  const int s = t * 16 + (lane & 15);
  act = s < ns;
  return act ? (int)s_slot_w[s] : lane;
}

// Gather a compacted sample's position and LOD level from its owner lane and
// encode it (4 lanes per sample, one level group each).
template <bool TAB16, bool PRECISE>
__device__ __forceinline__ void tile_encode(const FieldDev& F, const LevelDev* s_lv, __amdgpu_buffer_rsrc_t tab,
                                            int src, bool act, int lane, const float sx[3], float slst,
                                            float feat[8], uint32_t& fetches) {
  const float px[3] = {shfl_f(sx[0], src), shfl_f(sx[1], src), shfl_f(sx[2], src)};
  const float lstar = shfl_f(slst, src);
  encode_point<TAB16, PRECISE>(F, s_lv, tab, px, lstar, act, lane >> 4, feat, fetches);
}

// Per-ray SH values in FP32 for the FP32 path, laid out [lane][group g][i]
// with c = g + 4 i: a tile's lane group reads its four values in one 16-byte
// LDS load instead of evaluating all 16 polynomials of its sample's ray.
__device__ __forceinline__ void store_ray_sh_f32(const FieldDev& F, const Ray& r, float4* s_sh_lane) {
  float s[16];
  sh_basis16(r.dx, r.dy, r.dz, s);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = (uint32_t)(g + 4 * i) < F.nsh ? s[g + 4 * i] : 0.0f;
    s_sh_lane[g] = make_float4(v[0], v[1], v[2], v[3]);
  }
}

// Per-ray SH values in the MFMA element type, laid out [lane][group g][c = g + 4 i].
template <bool BF>
__device__ __forceinline__ void store_ray_sh(const FieldDev& F, const Ray& r, uint2* s_sh_lane) {
  float s[16];
  sh_basis16(r.dx, r.dy, r.dz, s);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = (uint32_t)(g + 4 * i) < F.nsh ? s[g + 4 * i] : 0.0f;
    s_sh_lane[g] = Half8<BF>::pack4(v);
  }
}

// Waves per SIMD the 16-bit kernels are compiled for (register budget
// 512 / waves).  4 measured fastest on the stereo C4 frame; 3 would let two
// tiles share each weight read but loses the latency cover of a fourth wave.
#ifndef VRN_WAVES16
#define VRN_WAVES16 4
#endif

template <bool TAB16, int MODE, int GEO>
__global__ __launch_bounds__(kF32Class<MODE> ? kBlockF32 : kBlock, kF32Class<MODE> ? 4 : VRN_WAVES16) void render_kernel(
    RenderArgs A) {
  constexpr int kThreads = kF32Class<MODE> ? kBlockF32 : kBlock;
  __shared__ __align__(16) uint8_t s_w[WeightSmem<MODE>::kBytes];
  __shared__ float s_b[kBiasTotal];
  __shared__ LevelDev s_lv[kMaxLevels];
  __shared__ uint32_t s_off[kMaxCams + 1];
  __shared__ uint32_t s_rb[kMaxCams], s_re[kMaxCams];
  __shared__ vrn_camera s_cams[kMaxCams];
  __shared__ uint32_t s_stats[kStats];
  // per-ray SH values: FP32 [lane][g] float4 (FP32 path) or packed 16-bit [lane][g] uint2
  __shared__ __align__(16) uint8_t s_sh_raw[kThreads * 4 * (kF32Class<MODE> ? 16 : 8)];
  uint2* s_sh = reinterpret_cast<uint2*>(s_sh_raw);
  float4* s_sh4 = reinterpret_cast<float4*>(s_sh_raw);
  __shared__ uint32_t s_slot[kThreads];
  // the FP32-class kernels keep their rays' steps per cell here between
  // marches, and with a sample table the neighbour pixel's direction (only a
  // found sample's LOD reads it): their registers run out (FP32X spilled 8 and
  // 19, now 2 and 14; 1024^2 unbounded frame 555 -> 527 us.  One more value of
  // the uniform lattice's rays changed nothing)
  __shared__ float s_ray[kF32Class<MODE> ? (GEO == 1 ? 6 : 3) * kThreads : 1];

  const FieldDev& F = A.F;
  const __amdgpu_buffer_rsrc_t tab = table_rsrc(F);
  if (threadIdx.x < F.L) s_lv[threadIdx.x] = F.levels[threadIdx.x];
  if (threadIdx.x < kStats) s_stats[threadIdx.x] = 0;
  const uint32_t tx = (A.W + kTile - 1) / kTile;
  const float inv_tx = 1.0f / (float)tx;
  // The cameras, from the caller's device memory or from the kernel's own
  // arguments, in words (the caller's need not be aligned to more).  In the
  // arguments they cost no copy ahead of the kernel (256^2 FP16 frame 66 ->
  // 63 us), and rays are set up from LDS (2x2048^2 FP32X house 5100 -> 5065).
  typedef const __attribute__((address_space(1))) uint32_t* GlobalWords;
  constexpr uint32_t kCamWords = sizeof(vrn_camera) / 4;
  const GlobalWords cams = (GlobalWords)(A.cams ? reinterpret_cast<uint64_t>(A.cams)
                                                : (uint64_t)__builtin_amdgcn_kernarg_segment_ptr() +
                                                      offsetof(RenderArgs, own_cams));
  uint32_t row_begin = 0, row_end = 0;
  if (threadIdx.x < A.n_cams) {
    row_begin = cams[threadIdx.x * kCamWords + offsetof(vrn_camera, row_begin) / 4];
    row_end = cams[threadIdx.x * kCamWords + offsetof(vrn_camera, row_end) / 4];
  }
  for (uint32_t i = threadIdx.x; i < A.n_cams * kCamWords; i += blockDim.x)
    reinterpret_cast<uint32_t*>(s_cams)[i] = cams[i];
  if (threadIdx.x < 64) {
    // camera c's first tile: an inclusive scan over the first 16 lanes
    uint32_t own = 0;
    if (threadIdx.x < A.n_cams) {
      const uint32_t rb = min(row_begin, A.H), re = min(max(row_end, rb), A.H);
      s_rb[threadIdx.x] = rb;
      s_re[threadIdx.x] = re;
      own = tx * ((re - rb + kTile - 1) / kTile);
    }
    uint32_t upto = own;
#pragma unroll
    for (int d = 1; d < kMaxCams; d *= 2) {
      const uint32_t o = (uint32_t)shfl_i((int)upto, lane_id() - d);
      if (lane_id() >= d) upto += o;
    }
    if (threadIdx.x < A.n_cams) s_off[threadIdx.x + 1] = upto;
    if (threadIdx.x == 0) s_off[0] = 0;
  }
  load_weights<MODE>(F, s_w, s_b);
  __syncthreads();

  const int lane = lane_id();
  const uint32_t n_tiles = s_off[A.n_cams];
  WsQueue* queues = reinterpret_cast<WsQueue*>(A.ws + kWsQueue);
  // Tiles go to the queues in runs of 2^run, each turn starting one queue
  // further, so that no queue is left with the same columns of every row.
  // 64 runs a frame balance the queues, and still leave an XCD's L2 whole tile
  // rows of a large frame (shorter runs cost the 2x2048^2 house frame 1 %).  A
  // queue's ids count its own tiles' pixels: the first dealt(q) go to its
  // blocks' waves by position, the rest to waves whose rays have all ended, as
  // does then what is left of the next two queues.  An atomic on a line that other XCDs share
  // takes some 20 ns, one after another: drawing every ray through them and
  // trying all eight queues at the end cost each launch 50-90 us (an empty
  // 512^2 frame 114 us, now 27).
  const uint32_t nq = gridDim.x >= (uint32_t)kQueues ? (uint32_t)kQueues : 1u, wpb = A.waves;
  const uint32_t run = n_tiles < 128u ? 0u : 25u - (uint32_t)__clz((int)n_tiles);
  const uint32_t size = ((((n_tiles + (1u << run) - 1u) >> run) + nq - 1u) / nq << run) * (kTile * kTile);
  auto dealt = [&](uint32_t i) { return (gridDim.x + nq - 1u - i) / nq * wpb * A.lanes; };
  uint32_t q = blockIdx.x % nq, tried = 0;
  bool dealing = true;

  Ray r;
  r.k = 0;
  r.k_hi = -1;
  r.lr = 0.0f;
  r.brick = -1;
  r.dist = 0;
  r.blo = r.bhi = 0u;
  r.delta = 0.0f;
  r.iq[0] = r.iq[1] = r.iq[2] = 0.0f;
  r.ox = r.oy = r.oz = r.dx = r.dy = r.dz = 0.0f;
  uint32_t pix = kNone, n = 0;
  float T = 1.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;
  uint32_t st_steps = 0, st_fetch = 0;                               // per lane
  uint32_t st_samples = 0, st_rays = 0, st_rounds = 0, st_tiles = 0;  // of the wave

  VRN_PHASE_START();
  auto retire = [&]() {
    float4 v = make_float4(cr, cg, cb, 1.0f - T);
    if (A.output != VRN_OUT_PQ) {
      v.x = pq_to_linear(v.x);
      v.y = pq_to_linear(v.y);
      v.z = pq_to_linear(v.z);
      if (A.output == VRN_OUT_SRGB) {
        v.x = srgb_oetf(v.x * A.exposure);
        v.y = srgb_oetf(v.y * A.exposure);
        v.z = srgb_oetf(v.z * A.exposure);
      }
    }
    VRN_DEBUG_COUNT((uint64_t)pix >= (uint64_t)A.n_cams * A.H * A.W, kDbgPixel);
    reinterpret_cast<float4*>(A.rgba)[pix] = v;
    if (A.nsamples) A.nsamples[pix] = n;
    pix = kNone;
  };

  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  while (wave < wpb) {
    // keep LDS reads of weights inside the loop (hoisting would pin the
    // weights in registers and drop occupancy to one wave per SIMD)
    asm volatile("" ::: "memory");
    VRN_PHASE(kPhComposite);
    // ---- 1. a wave whose rays have all ended takes the next ones ---------
    // (The rays of a tile take nearly the same number of samples, so lanes
    // filled one by one as they fell free gained no fuller MLP tiles, but one
    // refill a ray's end instead of one a tile: stereo 2x2048^2 house frame
    // 2.47 -> 2.37 ms, unbounded 1.88 -> 1.74, with thresholds of 16, 32, 48
    // and 56 free lanes in between.)
    while (__ballot(pix != kNone) == 0) {
      uint32_t base;
      if (dealing) {
        base = (blockIdx.x / nq * wpb + wave) * A.lanes;
        dealing = false;
      } else {
        base = dealt(q);
        uint32_t taken = 0;
        if (base < size) {
          if (lane == 0) taken = atomicAdd(&queues[q].taken, A.lanes);
          base += (uint32_t)__builtin_amdgcn_readfirstlane((int)taken);
        }
      }
      if (base >= size) {
        if (tried++ == kHelped) break;
        q = q + 1u == nq ? 0u : q + 1u;
        continue;
      }
      const uint32_t own = base / (kTile * kTile), turn = own >> run;
      const uint32_t tile = ((turn * nq + ((q + turn) & (nq - 1u))) << run) + (own & ((1u << run) - 1u));
      if (tile >= n_tiles) continue;
      uint32_t c = 0;
      while (c + 1 < A.n_cams && tile >= s_off[c + 1]) ++c;
      const uint32_t local = tile - s_off[c];
      // local / tx without an integer division: float quotient, then an exact
      // integer correction (local < 2^24)
      uint32_t ty = (uint32_t)((float)local * inv_tx);
      if (ty * tx > local) --ty;
      else if ((ty + 1) * tx <= local) ++ty;
      const uint32_t within = base % (kTile * kTile) + (uint32_t)lane;
      const uint32_t col = (local - ty * tx) * kTile + within % kTile;
      const uint32_t row = s_rb[c] + ty * kTile + within / kTile;
      if ((uint32_t)lane < A.lanes && col < A.W && row < s_re[c]) {
        setup_ray<GEO>(F, s_cams[c], col, row, r);
        if constexpr (kF32Class<MODE>) {
#pragma unroll
          for (int a = 0; a < 3; ++a) s_ray[a * kThreads + threadIdx.x] = r.iq[a];
          if constexpr (GEO == 1) {
            s_ray[3 * kThreads + threadIdx.x] = r.nx;
            s_ray[4 * kThreads + threadIdx.x] = r.ny;
            s_ray[5 * kThreads + threadIdx.x] = r.nz;
          }
        }
        if constexpr (!kF32Class<MODE>) store_ray_sh<MODE == 2>(F, r, &s_sh[threadIdx.x * 4]);
        else store_ray_sh_f32(F, r, &s_sh4[threadIdx.x * 4]);
        pix = (c * A.H + row) * A.W + col;
        T = 1.0f;
        cr = cg = cb = 0.0f;
        n = 0;
      }
      st_rays += (uint32_t)__popcll(__ballot(pix != kNone));
    }
    VRN_PHASE(kPhRefill);
    if (__ballot(pix != kNone) == 0) break;
    __builtin_amdgcn_wave_barrier();

    // ---- 2. march to the next evaluated sample ---------------------------
    int mres = 0;
    float st = 0.0f, sx[3] = {0.0f, 0.0f, 0.0f}, slst = 0.0f, sdt = F.dt;
    if (pix != kNone) {
      if constexpr (kF32Class<MODE>) {
#pragma unroll
        for (int a = 0; a < 3; ++a) r.iq[a] = s_ray[a * kThreads + threadIdx.x];
      }
      mres = march_next<GEO>(F, r, A.budget, st_steps, st, sx);
      if (mres == 2) retire();
      if (mres == 1) {
        if constexpr (kF32Class<MODE> && GEO == 1) {
          r.nx = s_ray[3 * kThreads + threadIdx.x];
          r.ny = s_ray[4 * kThreads + threadIdx.x];
          r.nz = s_ray[5 * kThreads + threadIdx.x];
        }
        if (F.lod) slst = (GEO == 1 && F.contract) ? level_star_contracted(F, r, st, sx) : level_star(F, st, r.lr);
        sdt = sample_step<GEO>(F, st);
      }
    }
    const bool has = mres == 1;
    const uint64_t m = __ballot(has);
    const int ns = __popcll(m);
    const int rank = __popcll(m & ((1ull << lane) - 1ull));
    const int nt = (ns + 15) >> 4;
    const int wave_base = (threadIdx.x >> 6) << 6;
    if (has) s_slot[wave_base + rank] = (uint32_t)lane;
    __builtin_amdgcn_wave_barrier();
    ++st_rounds;
    st_tiles += (uint32_t)nt;
    st_samples += (uint32_t)ns;

    VRN_PHASE(kPhMarch);
    // ---- 3. encode + MLP of the compacted samples -------------------------
    float so0 = 0.0f, sl0 = 0.0f, sl1 = 0.0f, sl2 = 0.0f;
    if constexpr (kF32Class<MODE>) {
      for (int t = 0; t < nt; ++t) {
        asm volatile("" ::: "memory");
        bool act;
        const int src = tile_source(&s_slot[wave_base], ns, t, lane, act);
        float feat[8], shs[4];
        tile_encode<TAB16, true>(F, s_lv, tab, src, act, lane, sx, slst, feat, st_fetch);
        {
          const float4 v = s_sh4[(wave_base + src) * 4 + (lane >> 4)];
          shs[0] = v.x;
          shs[1] = v.y;
          shs[2] = v.z;
          shs[3] = v.w;
        }
        VRN_PHASE(kPhEncode);
        float o0, lg[3];
        run_mlp<MODE>(s_w, s_b, F, feat, shs, lane, o0, lg);
        VRN_PHASE(kPhMlp);
        const int from = rank & 15;
        const float a0 = shfl_f(o0, from), a1 = shfl_f(lg[0], from);
        const float a2 = shfl_f(lg[1], from), a3 = shfl_f(lg[2], from);
        if (has && (rank >> 4) == t) {
          so0 = a0;
          sl0 = a1;
          sl1 = a2;
          sl2 = a3;
        }
        VRN_PHASE(kPhReturn);
      }
    } else {
      typedef Half8<MODE == 2> H;
      for (int t0 = 0; t0 < nt; t0 += kMlpBatch) {
        asm volatile("" ::: "memory");
        const int cnt = min(kMlpBatch, nt - t0);
        typename H::vec xin[kMlpBatch];
        uint2 shh[kMlpBatch];
#pragma unroll
        for (int t = 0; t < kMlpBatch; ++t)
          if (t < cnt) {
            bool act;
            const int src = tile_source(&s_slot[wave_base], ns, t0 + t, lane, act);
            if constexpr (TAB16 && MODE == 1) {
              const float px[3] = {shfl_f(sx[0], src), shfl_f(sx[1], src), shfl_f(sx[2], src)};
              uint32_t hf[4];
              encode_point_h2(F, s_lv, tab, px, shfl_f(slst, src), act, lane >> 4, hf, st_fetch);
              const uint4 u = make_uint4(hf[0], hf[1], hf[2], hf[3]);
              __builtin_memcpy(&xin[t], &u, 16);
            } else {
              float feat[8];
              tile_encode<TAB16, false>(F, s_lv, tab, src, act, lane, sx, slst, feat, st_fetch);
              xin[t] = H::pack(feat);
            }
            shh[t] = s_sh[(wave_base + src) * 4 + (lane >> 4)];
          }
        VRN_PHASE(kPhEncode);
        float o0[kMlpBatch], lg[kMlpBatch][3];
        // The 16-bit MFMA chain co-executes with other waves' VALU and gather
        // issue, so the batch runs at raised issue priority: its dependent
        // MFMAs then start as soon as their inputs are ready (0.5 % faster on
        // the stereo frame).  The FP32 MFMA does not co-execute and the FP32
        // path keeps the default priority (there the raise measured slower).
        __builtin_amdgcn_s_setprio(2);
        mlp_batch_16<MODE == 2, kMlpBatch>(reinterpret_cast<const uint4*>(s_w), s_b, cnt, xin, shh, lane, o0, lg);
        __builtin_amdgcn_s_setprio(0);
        VRN_PHASE(kPhMlp);
        const int from = rank & 15;
#pragma unroll
        for (int t = 0; t < kMlpBatch; ++t)
          if (t < cnt) {
            const float a0 = shfl_f(o0[t], from), a1 = shfl_f(lg[t][0], from);
            const float a2 = shfl_f(lg[t][1], from), a3 = shfl_f(lg[t][2], from);
            if (has && (rank >> 4) == t0 + t) {
              so0 = a0;
              sl0 = a1;
              sl1 = a2;
              sl2 = a3;
            }
          }
        VRN_PHASE(kPhReturn);
      }
    }

    // ---- 4. composite (FP32), terminate --------------------------------
    if (has) {
      VRN_DEBUG_COUNT(so0 != so0 || sl0 != sl0 || sl1 != sl1 || sl2 != sl2, kDbgMlpNaN);
      constexpr bool kFast = !kF32Class<MODE>;
      const float sd = comp_exp<kFast>(so0) * sdt;
      const float trans = comp_exp<kFast>(-sd);
      const float wgt = T * (1.0f - trans);
      cr = fmaf(wgt, sigmoidf<kFast>(sl0), cr);
      cg = fmaf(wgt, sigmoidf<kFast>(sl1), cg);
      cb = fmaf(wgt, sigmoidf<kFast>(sl2), cb);
      T = T * trans;
      ++n;
      if (T < F.t_min || n >= F.max_samples) retire();
    }
  }

  VRN_PHASE(kPhRefill);
  VRN_PHASE_FLUSH();
  atomicAdd(&s_stats[2], st_fetch);
  atomicAdd(&s_stats[3], st_steps);
  if (lane == 0) {
    atomicAdd(&s_stats[0], st_rays);
    atomicAdd(&s_stats[1], st_samples);
    atomicAdd(&s_stats[4], st_rounds);
    atomicAdd(&s_stats[5], st_tiles);
  }
  __syncthreads();
  if (dealt(nq - 1u) >= size) {
    // no queue was touched (a small launch): nothing to reset, only to count
    if (threadIdx.x < kStats)
      atomicAdd(reinterpret_cast<unsigned long long*>(A.ws + kWsStats) + threadIdx.x,
                (unsigned long long)s_stats[threadIdx.x]);
    return;
  }
  // Statistics and the count of finished blocks gather on the line of the
  // block's own queue, six lanes at once; its last block counts the queue as
  // finished, and the last of those adds the queues' sums up and leaves every
  // counter at zero.
  if (threadIdx.x < 64) {
    WsQueue& own = queues[blockIdx.x % nq];
    if (lane < kStats) atomicAdd(&own.stats[lane], (unsigned long long)s_stats[lane]);
    __threadfence();
    bool last = false;
    if (lane == 0 && atomicAdd(&own.done, 1u) == (gridDim.x + nq - 1u - blockIdx.x % nq) / nq - 1u) {
      __threadfence();
      last = atomicAdd(reinterpret_cast<uint32_t*>(A.ws + kWsDone), 1u) == nq - 1u;
    }
    if (__ballot(last) == 0) return;
    __threadfence();
    if (lane < kStats) {
      unsigned long long sum = 0;
      for (int i = 0; i < kQueues; ++i) sum += atomicExch(&queues[i].stats[lane], 0ull);
      atomicAdd(reinterpret_cast<unsigned long long*>(A.ws + kWsStats) + lane, sum);
    }
    if (lane < kQueues) {
      atomicExch(&queues[lane].taken, 0u);
      atomicExch(&queues[lane].done, 0u);
    }
    if (lane == 0) atomicExch(reinterpret_cast<uint32_t*>(A.ws + kWsDone), 0u);
    __threadfence();
  }
}

// ---------------------------------------------------------------------------
// stage kernels
// ---------------------------------------------------------------------------

__global__ void zero_kernel(uint32_t* p, uint64_t n_words) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n_words;
       i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

__global__ void rays_kernel(const vrn_camera* cams, uint32_t n_cams, uint32_t W, uint32_t H, float scale,
                            float* o, float* d, float* rr) {
  const uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
  if (i >= (uint64_t)n_cams * W * H) return;
  const uint32_t c = (uint32_t)(i / ((uint64_t)W * H));
  const uint32_t rem = (uint32_t)(i % ((uint64_t)W * H));
  const uint32_t row = rem / W, col = rem % W;
  float w[3], nn, dd[3];
  canonical_ray(cams[c], col, row, w, nn, dd);
  for (int a = 0; a < 3; ++a) {
    o[3 * i + a] = cams[c].c2w[4 * a + 3];
    d[3 * i + a] = dd[a];
  }
  rr[i] = cone_pitch(cams[c], w, nn, scale);
}

template <int GEO>
__global__ void march_kernel(FieldDev F, const vrn_camera* cams, uint32_t n_cams, uint32_t W, uint32_t H,
                             uint32_t* klist, uint32_t max_k, uint32_t* count) {
  const uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
  if (i >= (uint64_t)n_cams * W * H) return;
  const uint32_t c = (uint32_t)(i / ((uint64_t)W * H));
  const uint32_t rem = (uint32_t)(i % ((uint64_t)W * H));
  Ray r;
  setup_ray<GEO>(F, cams[c], rem % W, rem / W, r);
  uint32_t cnt = 0, steps = 0;
  float st, sx[3];
  while (cnt < F.max_samples) {
    if (march_next<GEO>(F, r, 0x40000000u, steps, st, sx) != 1) break;
    if (cnt < max_k) klist[i * max_k + cnt] = (uint32_t)(r.k - 1);
    ++cnt;
  }
  count[i] = cnt;
}

template <bool TAB16>
__global__ __launch_bounds__(kBlock) void encode_kernel(FieldDev F, const float* xyz, const float* tt,
                                                        const float* rr, uint32_t n, float* feat) {
  __shared__ LevelDev s_lv[kMaxLevels];
  if (threadIdx.x < F.L) s_lv[threadIdx.x] = F.levels[threadIdx.x];
  __syncthreads();
  const int lane = lane_id(), g = lane >> 4;
  const uint64_t p = (blockIdx.x * (uint64_t)(kBlock / 64) + threadIdx.x / 64) * 16 + (lane & 15);
  const bool act = p < n;
  float x[3] = {0.0f, 0.0f, 0.0f}, lstar = 0.0f;
  if (act) {
    for (int a = 0; a < 3; ++a) x[a] = xyz[3 * p + a];
    if (F.lod) lstar = level_star(F, tt[p], logf(rr[p]) + F.lod_c);
  }
  float f[8];
  uint32_t fetches = 0;
  encode_point<TAB16, true>(F, s_lv, table_rsrc(F), x, lstar, act, g, f, fetches);
  if (!act) return;
  for (int j = 0; j < 4; ++j) {
    const int lev = g + 4 * j;
    if (lev < (int)F.L) {
      feat[p * (2 * F.L) + 2 * lev] = f[2 * j];
      feat[p * (2 * F.L) + 2 * lev + 1] = f[2 * j + 1];
    }
  }
}

// Blocks stay and walk the samples a tile a wave at a time, so that a block's
// weights are staged once; a wave loads its next tile's inputs before it
// evaluates the present one.  2 M samples of 16 levels, FP16: 183 us with a
// block staging its weights for every 64 samples, 105 with resident blocks, 96
// with the loads ahead, of which the reads and writes take 64 at the rate of a
// copy and the LDS reads of weights and biases 58.  (Two tiles a wave halve
// the latter, but at 82 registers fewer waves hide the loads: 133 us.  Blocks
// of 256 and 1024 threads: 101 and 98.)  FP32X 487 -> 234 us; FP32 416 -> 338,
// bound by its MFMA (245 us).
template <int MODE>
__global__ __launch_bounds__(kMlpThreads) void mlp_kernel(FieldDev F, const float* feat, const float* dir, uint32_t n,
                                                          float* sigma, float* rgb) {
  __shared__ __align__(16) uint8_t s_w[WeightSmem<MODE>::kBytes];
  __shared__ float s_b[kBiasTotal];
  load_weights<MODE>(F, s_w, s_b);
  __syncthreads();
  const int lane = lane_id(), g = lane >> 4;
  const uint32_t tiles = mlp_tiles(n), wpb = blockDim.x / 64u;
  float f[8], d[3];
  auto load = [&](uint32_t t) {
    const uint64_t p = (uint64_t)t * 16u + (uint32_t)(lane & 15);
    const bool act = p < n;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int lev = g + 4 * j;
      float2 v = make_float2(0.0f, 0.0f);
      if (act && lev < (int)F.L) __builtin_memcpy(&v, feat + p * (2 * F.L) + 2 * lev, 8);   // 4-byte aligned
      f[2 * j] = v.x;
      f[2 * j + 1] = v.y;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) d[a] = act ? dir[3 * p + a] : 0.0f;
  };
  uint32_t t = blockIdx.x * wpb + threadIdx.x / 64u;
  if (t < tiles) load(t);
  while (t < tiles) {
    float shs[4], now[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) now[i] = f[i];
    sh_select(F, d[0], d[1], d[2], g, shs);
    const uint64_t p = (uint64_t)t * 16u + (uint32_t)(lane & 15);
    t += gridDim.x * wpb;
    if (t < tiles) load(t);
    asm volatile("" ::: "memory");
    float o0, lg[3];
    run_mlp<MODE>(s_w, s_b, F, now, shs, lane, o0, lg);
    // lanes 0..15 hold the results: one output a lane group, so that one
    // library exponential serves all four
    const float z0 = shfl_f(lg[0], lane & 15), z1 = shfl_f(lg[1], lane & 15), z2 = shfl_f(lg[2], lane & 15);
    const float e = expf(g == 0 ? o0 : -(g == 1 ? z0 : g == 2 ? z1 : z2));
    if (p < n) {
      if (g == 0) sigma[p] = e;
      else rgb[3 * p + (uint32_t)(g - 1)] = __builtin_amdgcn_rcpf(1.0f + e);
    }
  }
}

// ---------------------------------------------------------------------------
// grid pruning (Sec. 4.3, App. C): max opacity over points inside each
// occupied voxel, threshold alpha; pruning only clears bits.
//
// Three launches: (1) the output bits start as the field's occupancy (and
// the maximum opacity, by a launch of its own, as NaN); (2) the non-empty
// groups of four bricks along x are listed with their places in the order of
// all occupied voxels; (3) persistent waves take chunks of that order, look
// the chunk's first group up, gather its voxels row by row in LDS and
// evaluate them -- 16-sample MFMA tiles through the same encode and density
// layers as the renderer -- then clear the bits of voxels below alpha.  Only
// occupied voxels cost work, and the weights are staged once per resident
// block.
//
// What bounds it is the fabric behind the L2s: on the 512^3 house field (4.0 M
// voxels x 4 points x 16 levels) the finer levels' corners miss L2, a
// 128-byte line each, at 7.5 TB/s; the FP32 and FP16 MLPs take the same time.
// The hash keeps the 32 cells of an aligned run along x in one line, so what
// shares lines is neighbours along x and, on the coarser levels, all
// neighbours, if they are looked up at about the same time: the L2 has room
// for some 40 lines a wave.  A tile is therefore the same point of up to 16
// voxels along x, where they form runs, and the waves of an XCD take neighbouring chunks of 16 side
// by side.  FP16, 4 points: 6.40 ms with whole bricks dealt to the waves of all
// XCDs in turn and four points of four voxels a tile, 6.05 ms with one
// contiguous share a wave, 5.72, 5.60 and 5.40 ms with chunks of 64, 32 and 16
// voxels (8 points: 9.36 -> 6.49 ms).  Other cache policies of the gathers cost
// 4 % (device scope) to 50 % (non-temporal).
// ---------------------------------------------------------------------------

__device__ __forceinline__ bool cell_occupied(const FieldDev& F, uint32_t x, uint32_t y, uint32_t z) {
  const uint32_t b = (x >> 2) + F.Gb * ((y >> 2) + F.Gb * (z >> 2));
  const unsigned long long w = F.bricks[b];
  return (w >> ((x & 3) + 4 * (y & 3) + 16 * (z & 3))) & 1ull;
}

// offsets of point i inside a voxel: 4 = tetrahedral corners of the 2x2x2
// sub-lattice at {1/4, 3/4}; otherwise a p^3 grid at (i + 1/2) / p
__device__ __forceinline__ float voxel_offset(uint32_t npts, uint32_t p, uint32_t i, int axis) {
  if (npts == 4) {
    const float q = 0.25f, t = 0.75f;
    const float tab[4][3] = {{q, q, q}, {t, t, q}, {t, q, t}, {q, t, t}};
    return tab[i & 3][axis];
  }
  const uint32_t c = axis == 0 ? i % p : (axis == 1 ? (i / p) % p : i / (p * p));
  return ((float)c + 0.5f) / (float)p;
}

// (1) one thread per 32-bit output word (G^3 < 2^31, so 32-bit indices)
__global__ void prune_init_kernel(FieldDev F, uint32_t* bits_out) {
  const uint32_t G = F.G;
  const uint32_t n = G * G * G;
  const uint32_t w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= (n + 31u) / 32u) return;
  const uint32_t i0 = w * 32u;
  uint32_t x = i0 % G, y = (i0 / G) % G, z = i0 / (G * G);
  if ((G & 31u) == 0u) {
    // the word is one row of 32 cells at fixed (y, z): 4 cells from each of
    // 8 bricks, taken from the brick words directly
    const uint32_t shift = 4u * (y & 3u) + 16u * (z & 3u);
    const uint32_t b0 = (x >> 2) + F.Gb * ((y >> 2) + F.Gb * (z >> 2));
    uint32_t out = 0u;
#pragma unroll
    for (uint32_t k = 0; k < 8u; ++k) out |= (uint32_t)((F.bricks[b0 + k] >> shift) & 0xFull) << (4u * k);
    bits_out[w] = out;
    return;
  }
  uint32_t out = 0u;
  for (uint32_t j = 0; j < 32u && i0 + j < n; ++j) {
    if (cell_occupied(F, x, y, z)) out |= 1u << j;
    if (++x == G) {
      x = 0;
      if (++y == G) {
        y = 0;
        ++z;
      }
    }
  }
  bits_out[w] = out;
}

// the maximum opacity of every voxel starts as NaN; the occupied ones are
// written by the pass (at 512^3 a write stream of 0.5 GB; together with the
// bits, a thread a word, it took 1.6 ms)
__global__ void nan_kernel(float* p, uint64_t n) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = __builtin_nanf("");
}

// (2) the non-empty groups of four bricks along x, nearly in order: x the
// index gx + ngx (by + Gb bz) with ngx = ceil(Gb / 4), y the number of
// occupied voxels of the groups listed before.  total (zeroed before): groups
// in the high word, voxels in the low one.  (Two replayed passes that run at
// once may count every group twice: no slot beyond the list is written.)
__global__ void group_list_kernel(FieldDev F, uint2* list, unsigned long long* total) {
  const uint32_t ngx = (F.Gb + 3u) / 4u, n = ngx * F.Gb * F.Gb;
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t voxels = 0;
  if (i < n) {
    const uint32_t gx = i % ngx, row = i / ngx, b = row * F.Gb + 4u * gx;
    for (uint32_t j = 0; j < 4u && 4u * gx + j < F.Gb; ++j) voxels += (uint32_t)__popcll(F.bricks[b + j]);
  }
  const uint64_t m = __ballot(voxels != 0u);
  if (m == 0) return;
  const int lane = lane_id();
  uint32_t upto = voxels;
#pragma unroll
  for (int d = 1; d < 64; d *= 2) {
    const uint32_t o = (uint32_t)shfl_i((int)upto, lane - d);
    if (lane >= d) upto += o;
  }
  unsigned long long base = 0;
  if (lane == 63) base = atomicAdd(total, (unsigned long long)__popcll(m) << 32 | upto);
  const uint32_t entry = (uint32_t)__builtin_amdgcn_readlane((int)(base >> 32), 63);
  const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)base, 63);
  const uint32_t slot = entry + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
  if (voxels != 0u && slot < n) list[slot] = make_uint2(i, before + upto - voxels);
}

// Density layers only (the pruning pass needs sigma, not color), in the
// renderer's fragment layout.  Lanes 0..15 return the density pre-activation
// o0 of samples 0..15.
__device__ __forceinline__ float density_tile_f32(const float4* __restrict__ sw, const float* __restrict__ sb,
                                                  uint32_t d1_groups, const float feat[8], int lane) {
  const int g = lane >> 4;
  v4f h[4];
#pragma unroll
  for (int ot = 0; ot < 4; ++ot) h[ot] = bias_acc(sb, kB1 + 16 * ot, g);
#pragma unroll
  for (int s4 = 0; s4 < 2; ++s4) {
    if ((uint32_t)s4 < d1_groups) {
#pragma unroll
      for (int ot = 0; ot < 4; ++ot) {
        const float4 w = sw[kW32_D1 / 4 + (ot * 2 + s4) * 64 + lane];
        h[ot] = mfma_f32(w.x, feat[4 * s4 + 0], h[ot]);
        h[ot] = mfma_f32(w.y, feat[4 * s4 + 1], h[ot]);
        h[ot] = mfma_f32(w.z, feat[4 * s4 + 2], h[ot]);
        h[ot] = mfma_f32(w.w, feat[4 * s4 + 3], h[ot]);
      }
    }
  }
#pragma unroll
  for (int ot = 0; ot < 4; ++ot) h[ot] = relu4(h[ot]);
  v4f o = zero4();
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const float4 w = sw[kW32_D2 / 4 + it * 64 + lane];
    o = mfma_f32(w.x, h[it][0], o);
    o = mfma_f32(w.y, h[it][1], o);
    o = mfma_f32(w.z, h[it][2], o);
    o = mfma_f32(w.w, h[it][3], o);
  }
  return o[0] + sb[kB2 + 4 * g];
}

template <bool BF>
__device__ __forceinline__ float density_tile_16(const uint4* __restrict__ sw, const float* __restrict__ sb,
                                                 const float feat[8], int lane) {
  typedef Half8<BF> H;
  typedef typename H::vec vec;
  const int g = lane >> 4;
  auto wfrag = [&](int off16, int idx) -> vec {
    const uint4 u = sw[off16 / 8 + idx * 64 + lane];
    vec v;
    __builtin_memcpy(&v, &u, 16);
    return v;
  };
  const vec xin = H::pack(feat);
  vec hp[2];
#pragma unroll
  for (int pair = 0; pair < 2; ++pair) {
    const v4f a = H::mfma(wfrag(kW16_D1, 2 * pair), xin, bias_acc(sb, kB1 + 32 * pair, g));
    const v4f b = H::mfma(wfrag(kW16_D1, 2 * pair + 1), xin, bias_acc(sb, kB1 + 32 * pair + 16, g));
    const float hv[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    hp[pair] = H::relu_pack(hv);
  }
  const v4f o = H::mfma(wfrag(kW16_D2, 1), hp[1], H::mfma(wfrag(kW16_D2, 0), hp[0], bias_acc(sb, kB2, g)));
  return o[0];
}

// Density layers by split BF16 (mode 3): the D1 and D2 fragments of each
// of the three parts, staged [part][kW16_C1].
__device__ __forceinline__ float density_tile_x3(const uint4* __restrict__ sw3, const float* __restrict__ sb,
                                                 const float feat[8], int lane) {
  const int g = lane >> 4;
  const Bf3 xin = split_bf3(feat);
  float hv[16];
#pragma unroll
  for (int ot = 0; ot < 4; ++ot) {
    const v4f h = relu4(mfma_bf3(wfrag_bf3(sw3, kW16_C1, kW16_D1, ot, lane), xin, bias_acc(sb, kB1 + 16 * ot, g)));
#pragma unroll
    for (int r = 0; r < 4; ++r) hv[4 * ot + r] = h[r];
  }
  v4f o = mfma_bf3(wfrag_bf3(sw3, kW16_C1, kW16_D2, 0, lane), split_bf3(hv), zero4());
  o = mfma_bf3(wfrag_bf3(sw3, kW16_C1, kW16_D2, 1, lane), split_bf3(hv + 8), o);
  return o[0] + sb[kB2 + 4 * g];
}

// The density-layer weights (D1 and D2) are the first kW32_C1 / kW16_C1
// elements of each weight form (of each of the three parts in mode 3).
template <int MODE>
struct DensitySmem {
  static constexpr int kBytes = (MODE == 0) ? kW32_C1 * 4 : (MODE == 3 ? 3 * kW16_C1 * 2 : kW16_C1 * 2);
};

constexpr uint32_t kPruneChunk = 16;   // most voxels a wave takes at once

// (3) persistent pruning waves over the group list.  The list is the field's,
// not the call's: where replayed calls on one field overlap it may hold
// anything, so nothing taken from it reaches an address unchecked.
template <bool TAB16, int MODE>
__global__ __launch_bounds__(kBlock) void prune_kernel(FieldDev F, float alpha, uint32_t npts, uint32_t p,
                                                      const uint2* list, const unsigned long long* total,
                                                      uint32_t* bits_out, float* max_op) {
  __shared__ __align__(16) uint8_t s_w[DensitySmem<MODE>::kBytes];
  __shared__ float s_b[kBiasTotal];
  __shared__ LevelDev s_lv[kMaxLevels];
  __shared__ uint32_t s_q[kBlock / 64][kPruneChunk];
  {
    const uint4* src = weight_src<MODE>(F);
    uint4* dst = reinterpret_cast<uint4*>(s_w);
    if constexpr (MODE == 3) {
      constexpr int kPart = kW16_C1 * 2 / 16;   // uint4 per part
      for (int i = threadIdx.x; i < 3 * kPart; i += blockDim.x)
        dst[i] = src[(i / kPart) * (kW16Total * 2 / 16) + i % kPart];
    } else {
      for (int i = threadIdx.x; i < DensitySmem<MODE>::kBytes / 16; i += blockDim.x) dst[i] = src[i];
    }
    for (int i = threadIdx.x; i < kBiasTotal; i += blockDim.x) s_b[i] = F.bias[i];
    if (threadIdx.x < F.L) s_lv[threadIdx.x] = F.levels[threadIdx.x];
  }
  __syncthreads();
  const __amdgpu_buffer_rsrc_t tab = table_rsrc(F);
  const int lane = lane_id(), g = lane >> 4, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  uint32_t* q = s_q[wv];
  // Each XCD takes an eighth of the voxels, in list order, and its waves one
  // chunk of it after the other side by side, so that neighbours meet in one L2.
  const uint32_t nx = gridDim.x >= (uint32_t)kQueues ? (uint32_t)kQueues : 1u, xcd = blockIdx.x % nx;
  const uint32_t G = F.G, Gb = F.Gb, ngx = (Gb + 3u) / 4u, n_groups = ngx * Gb * Gb;
  const unsigned long long totals = *total;
  const uint32_t n_list = min((uint32_t)(totals >> 32), n_groups), n_vox = min((uint32_t)totals, G * G * G);
  const uint32_t start = (uint32_t)((uint64_t)n_vox * xcd / nx), stop = (uint32_t)((uint64_t)n_vox * (xcd + 1u) / nx);
  const uint32_t waves = (gridDim.x + nx - 1u - xcd) / nx * (kBlock / 64), share = (stop - start + waves - 1u) / waves;
  // A wave takes 16 voxels at once; where there are fewer for each, so many that
  // every wave has some, in whole tiles of a run (100 voxels of 64 points on
  // seven of 6144 waves 200 us, on a hundred 44; 10,000 of 4 points 99 and 84).
  const uint32_t row = npts == 4u ? 1u : p, full = 16u / row;
  const uint32_t chunk = share <= full ? max(share, 1u) : share <= 2u * full ? min(2u * full, kPruneChunk) : kPruneChunk;
  const uint32_t stride = waves * chunk;
  const float cell = F.inv_cs;
  for (uint32_t begin = start + (blockIdx.x / nx * (kBlock / 64) + (uint32_t)wv) * chunk; begin < stop; begin += stride) {
    const uint32_t end = min(begin + chunk, stop);
    uint32_t i = 0;                     // the last entry that starts at or before begin
    for (uint32_t hi = n_list; hi - i > 1u;) {
      const uint32_t mid = i + (hi - i) / 2u;
      if (list[mid].y <= begin) i = mid;
      else hi = mid;
    }
    if (lane < (int)kPruneChunk) q[lane] = kNone;
    // (every group holds a voxel: a chunk meets no more groups than it has voxels)
    for (const uint32_t past = min(i + kPruneChunk, n_list); i < past; ++i) {
      const uint2 entry = list[i];
      if (entry.y >= end || entry.x >= n_groups) break;
      // queue the occupied voxels of one group, rows of 16 along x one after
      // another, packed x | y << 10 | z << 20; lane 4 r + j holds row r of
      // brick j
      const uint32_t e = entry.x, j = (uint32_t)lane & 3u, r = (uint32_t)lane >> 2;
      const uint32_t bx = 4u * (e % ngx) + j, by = (e / ngx) % Gb, bz = e / (ngx * Gb);
      const uint32_t four = bx < Gb ? (uint32_t)(F.bricks[bx + Gb * (by + Gb * bz)] >> (4u * r)) & 15u : 0u;
      uint32_t at = entry.y;            // place of the lane's first voxel in list order
#pragma unroll
      for (uint32_t k = 0; k < 4u; ++k) {
        const uint64_t m = __ballot((four >> k) & 1u);
        at += (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
      }
      const uint32_t v = (4u * bx) | ((4u * by + (r & 3u)) << 10) | ((4u * bz + (r >> 2)) << 20);
#pragma unroll
      for (uint32_t k = 0; k < 4u; ++k)
        if ((four >> k) & 1u) {
          if (at >= begin && at < end) q[at - begin] = v + k;
          ++at;
        }
    }
    __builtin_amdgcn_wave_barrier();
    // How many points of a voxel stand side by side in a tile: of runs of voxels
    // along x one, or the p along x of p^3 patterns, so that the voxels of a run
    // meet; of voxels apart from each other (runs of 1.25 or less, where the two
    // measure the same), and where a small chunk leaves lanes free, as many as
    // fit.  4 points: planes across x 612 -> 555 us, along x 322 with one point
    // and 380 with four; 120,000 scattered voxels 564 -> 490; the 256^3 room
    // 1100 -> 998.
    const int V = (int)(end - begin);
    const uint64_t joined = __ballot(lane > 0 && lane < V && q[lane & 15] == q[(lane - 1) & 15] + 1u);
    const bool apart = 5u * (uint32_t)__popcll(joined) <= (uint32_t)V;
    const uint32_t side = min(npts, apart ? 16u : max(row, 16u / (uint32_t)V));
    const uint32_t vpt = 16u / side;
    const uint32_t vl = ((uint32_t)lane & 15u) / side, px = ((uint32_t)lane & 15u) - vl * side;
    for (int t = 0; t < V; t += (int)vpt) {
      const int vr = t + (int)vl;
      const uint32_t c = q[vl < vpt && vr < V ? vr : 0];
      const bool act = vl < vpt && vr < V && c != kNone;
      const uint32_t cc[3] = {c & 1023u, (c >> 10) & 1023u, c >> 20};
      float most = 0.0f;
      // (all lanes take every turn: a matrix product reads its weights from all)
      for (uint32_t first = 0; first < npts; first += side) {
        asm volatile("" ::: "memory");
        const uint32_t pi = first + px;
        float x[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) x[a] = F.amin[a] + ((float)cc[a] + voxel_offset(npts, p, pi, a)) * cell;
        float feat[8];
        uint32_t fetches = 0;
        // every level weighs 1 (no ray, no LOD): L* above the finest level
        encode_point<TAB16, kF32Class<MODE>>(F, s_lv, tab, x, 1.0e9f, act && pi < npts, g, feat, fetches);
        float o0;
        if constexpr (MODE == 0)
          o0 = density_tile_f32(reinterpret_cast<const float4*>(s_w), s_b, F.d1_ksteps / 4, feat, lane);
        else if constexpr (MODE == 3)
          o0 = density_tile_x3(reinterpret_cast<const uint4*>(s_w), s_b, feat, lane);
        else
          o0 = density_tile_16<MODE == 2>(reinterpret_cast<const uint4*>(s_w), s_b, feat, lane);
        float op = 1.0f - expf(-expf(o0) * F.dt);
        // a NaN opacity (16-bit activations that overflowed) keeps the voxel
        if (!(op == op)) op = 1.0f;
        if (pi < npts) most = fmaxf(most, op);
      }
      float top = most;
      for (uint32_t k = 1; k < side; ++k) top = fmaxf(top, shfl_f(most, lane + (int)k));
      if (act && g == 0 && px == 0u) {
        const uint32_t idx = cc[0] + G * (cc[1] + G * cc[2]);
        if (!(top >= alpha)) atomicAnd(&bits_out[idx >> 5], ~(1u << (idx & 31u)));
        if (max_op) max_op[idx] = top;
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Rebuild a resident field's bricks from linear bits.  With the distances
// below 97 us at 512^3, where bricks by single cells and a coarse grid and its
// dilation by a few serial threads took 700 us.
__global__ void bricks_from_bits_kernel(FieldDev F, unsigned long long* bricks, const uint32_t* bits) {
  const uint64_t b = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
  const uint64_t nb = (uint64_t)F.Gb * F.Gb * F.Gb;
  if (b >= nb) return;
  const uint32_t bx = (uint32_t)(b % F.Gb), by = (uint32_t)((b / F.Gb) % F.Gb), bz = (uint32_t)(b / ((uint64_t)F.Gb * F.Gb));
  unsigned long long w = 0ull;
  if ((F.G & 3u) == 0u) {
    // four cells of a row lie in one word: 16 loads, not 64
#pragma unroll
    for (uint32_t r = 0; r < 16; ++r) {
      const uint64_t idx = 4 * bx + (uint64_t)F.G * (4 * by + (r & 3) + (uint64_t)F.G * (4 * bz + (r >> 2)));
      w |= (unsigned long long)((bits[idx >> 5] >> (idx & 31)) & 15u) << (4 * r);
    }
    bricks[b] = w;
    return;
  }
  for (uint32_t i = 0; i < 64; ++i) {
    const uint32_t x = 4 * bx + (i & 3), y = 4 * by + ((i >> 2) & 3), z = 4 * bz + (i >> 4);
    if (x < F.G && y < F.G && z < F.G) {
      const uint64_t idx = x + (uint64_t)F.G * (y + (uint64_t)F.G * z);
      if ((bits[idx >> 5] >> (idx & 31)) & 1u) w |= 1ull << i;
    }
  }
  bricks[b] = w;
}

// Chebyshev distance in bricks to the nearest non-empty one (at most kMaxDist),
// one axis a launch: d'(i) = min over j of max(|j - i|, d(i + j)), searched
// outwards and stopped at the best so far, which a step further out cannot
// beat.  The first pass reads the bricks themselves.  (Directional distances,
// one per octant, would save another 5 % of the march's tests for eight times
// the memory.)
template <int AXIS>
__global__ void brick_distance_kernel(FieldDev F, const uint8_t* in, uint8_t* out) {
  const uint32_t Gb = F.Gb, i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= Gb * Gb * Gb) return;
  auto at = [&](uint32_t b) -> int {
    if constexpr (AXIS == 0) return F.bricks[b] != 0ull ? 0 : kMaxDist;
    else return in[b];
  };
  const int c = (int)(AXIS == 0 ? i % Gb : AXIS == 1 ? (i / Gb) % Gb : i / (Gb * Gb));
  const uint32_t pitch = AXIS == 0 ? 1u : AXIS == 1 ? Gb : Gb * Gb;
  int best = at(i);
  for (int j = 1; j < best; ++j) {
    int v = kMaxDist;
    if (c >= j) v = at(i - (uint32_t)j * pitch);
    if (c + j < (int)Gb) v = min(v, at(i + (uint32_t)j * pitch));
    best = min(best, max(j, v));
    if (c < j && c + j >= (int)Gb) break;
  }
  out[i] = (uint8_t)best;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

template <bool TAB16, int MODE, int GEO>
static int blocks_per_cu_impl() {
  static int cached = -1;
  if (cached < 0) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, render_kernel<TAB16, MODE, GEO>,
                                                     render_block_threads(MODE), 0) !=
            hipSuccess ||
        nb < 1)
      nb = 1;
    cached = nb;
  }
  return cached;
}

template <int GEO>
static int blocks_per_cu_geo(int table_f16, int compute) {
  if (table_f16) {
    if (compute == 0) return blocks_per_cu_impl<true, 0, GEO>();
    if (compute == 1) return blocks_per_cu_impl<true, 1, GEO>();
    if (compute == 3) return blocks_per_cu_impl<true, 3, GEO>();
    return blocks_per_cu_impl<true, 2, GEO>();
  }
  if (compute == 0) return blocks_per_cu_impl<false, 0, GEO>();
  if (compute == 1) return blocks_per_cu_impl<false, 1, GEO>();
  if (compute == 3) return blocks_per_cu_impl<false, 3, GEO>();
  return blocks_per_cu_impl<false, 2, GEO>();
}

int render_blocks_per_cu(const FieldDev& F, int compute) {
  return F.lat ? blocks_per_cu_geo<1>(F.table_f16, compute) : blocks_per_cu_geo<0>(F.table_f16, compute);
}

template <int GEO>
static void launch_render_geo(const RenderArgs& a, int compute, dim3 gr, dim3 bl, hipStream_t s) {
  if (a.F.table_f16) {
    if (compute == 0) hipLaunchKernelGGL((render_kernel<true, 0, GEO>), gr, bl, 0, s, a);
    else if (compute == 1) hipLaunchKernelGGL((render_kernel<true, 1, GEO>), gr, bl, 0, s, a);
    else if (compute == 3) hipLaunchKernelGGL((render_kernel<true, 3, GEO>), gr, bl, 0, s, a);
    else hipLaunchKernelGGL((render_kernel<true, 2, GEO>), gr, bl, 0, s, a);
  } else {
    if (compute == 0) hipLaunchKernelGGL((render_kernel<false, 0, GEO>), gr, bl, 0, s, a);
    else if (compute == 1) hipLaunchKernelGGL((render_kernel<false, 1, GEO>), gr, bl, 0, s, a);
    else if (compute == 3) hipLaunchKernelGGL((render_kernel<false, 3, GEO>), gr, bl, 0, s, a);
    else hipLaunchKernelGGL((render_kernel<false, 2, GEO>), gr, bl, 0, s, a);
  }
}

hipError_t launch_render(const RenderArgs& a, int compute, int grid, int threads, hipStream_t s) {
  const dim3 gr(grid), bl(threads);
  if (a.F.lat) launch_render_geo<1>(a, compute, gr, bl, s);
  else launch_render_geo<0>(a, compute, gr, bl, s);
  return hipGetLastError();
}

template <bool TAB16, int MODE>
static void launch_prune_mode(const FieldDev& F, float alpha, uint32_t npts, uint32_t p, uint32_t* bits_out,
                              float* max_op, int n_cu, hipStream_t s) {
  static int per_cu = -1;
  if (per_cu < 0) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, prune_kernel<TAB16, MODE>, kBlock, 0) != hipSuccess || nb < 1)
      nb = 1;
    per_cu = nb;
  }
  hipLaunchKernelGGL((prune_kernel<TAB16, MODE>), dim3((unsigned)(per_cu * n_cu)), dim3(kBlock), 0, s, F, alpha, npts,
                     p, F.group_list, F.group_total, bits_out, max_op);
}

hipError_t launch_prune(const FieldDev& F, float alpha, uint32_t npts, int compute, uint32_t* bits_out,
                        float* max_op, int n_cu, hipStream_t s) {
  uint32_t p = 1;
  while ((p + 1) * (p + 1) * (p + 1) <= npts) ++p;
  const uint32_t n = F.G * F.G * F.G;
  const uint32_t words = (n + 31u) / 32u;
  hipLaunchKernelGGL(prune_init_kernel, dim3((words + 255u) / 256u), dim3(256), 0, s, F, bits_out);
  if (max_op) hipLaunchKernelGGL(nan_kernel, dim3(std::min((n + 255u) / 256u, (uint32_t)n_cu * 32u)), dim3(256), 0, s, max_op, (uint64_t)n);
  hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(64), 0, s,
                     reinterpret_cast<uint32_t*>(F.group_total), (uint64_t)2);
  const uint32_t ng = (F.Gb + 3u) / 4u * F.Gb * F.Gb;
  hipLaunchKernelGGL(group_list_kernel, dim3((ng + 255u) / 256u), dim3(256), 0, s, F, F.group_list, F.group_total);
  if (F.table_f16) {
    if (compute == 0) launch_prune_mode<true, 0>(F, alpha, npts, p, bits_out, max_op, n_cu, s);
    else if (compute == 1) launch_prune_mode<true, 1>(F, alpha, npts, p, bits_out, max_op, n_cu, s);
    else if (compute == 3) launch_prune_mode<true, 3>(F, alpha, npts, p, bits_out, max_op, n_cu, s);
    else launch_prune_mode<true, 2>(F, alpha, npts, p, bits_out, max_op, n_cu, s);
  } else {
    if (compute == 0) launch_prune_mode<false, 0>(F, alpha, npts, p, bits_out, max_op, n_cu, s);
    else if (compute == 1) launch_prune_mode<false, 1>(F, alpha, npts, p, bits_out, max_op, n_cu, s);
    else if (compute == 3) launch_prune_mode<false, 3>(F, alpha, npts, p, bits_out, max_op, n_cu, s);
    else launch_prune_mode<false, 2>(F, alpha, npts, p, bits_out, max_op, n_cu, s);
  }
  return hipGetLastError();
}

// Launched through the calls that return a launch's own status: the thread's
// last error may be another call's, and loading a field does not fail for it.
hipError_t launch_brick_distance(const FieldDev& F, hipStream_t s) {
  const dim3 gr((F.Gb * F.Gb * F.Gb + 255u) / 256u), bl(256);
  FieldDev f = F;
  uint8_t *d = const_cast<uint8_t*>(F.dist), *tmp = reinterpret_cast<uint8_t*>(F.group_list);
  const uint8_t *none = nullptr, *from_d = d, *from_tmp = tmp;
  void *x[] = {&f, &none, &d}, *y[] = {&f, &from_d, &tmp}, *z[] = {&f, &from_tmp, &d};
  hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(&brick_distance_kernel<0>), gr, bl, x, 0, s);
  if (e == hipSuccess) e = hipLaunchKernel(reinterpret_cast<const void*>(&brick_distance_kernel<1>), gr, bl, y, 0, s);
  if (e == hipSuccess) e = hipLaunchKernel(reinterpret_cast<const void*>(&brick_distance_kernel<2>), gr, bl, z, 0, s);
  return e;
}

hipError_t launch_set_occupancy(const FieldDev& F, const uint32_t* bits, hipStream_t s) {
  const uint64_t nb = (uint64_t)F.Gb * F.Gb * F.Gb;
  hipLaunchKernelGGL(bricks_from_bits_kernel, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, s, F,
                     const_cast<unsigned long long*>(F.bricks), bits);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? launch_brick_distance(F, s) : e;
}

hipError_t phase_cycles(unsigned long long out[kPhaseSlots], bool reset) {
#ifdef VRN_PHASE_TIMING
  hipError_t e = hipMemcpyFromSymbol(out, HIP_SYMBOL(vrn_phase_cycles), sizeof(unsigned long long) * kPhaseSlots);
  if (e == hipSuccess && reset) {
    const unsigned long long zero[kPhaseSlots] = {};
    e = hipMemcpyToSymbol(HIP_SYMBOL(vrn_phase_cycles), zero, sizeof(zero));
  }
  return e;
#else
  (void)out;
  (void)reset;
  return hipErrorNotSupported;
#endif
}

hipError_t debug_counters(unsigned long long out[kDbgSlots], bool reset) {
#ifdef VRN_DEBUG_CHECKS
  hipError_t e = hipMemcpyFromSymbol(out, HIP_SYMBOL(vrn_debug_counts), sizeof(unsigned long long) * kDbgSlots);
  if (e == hipSuccess && reset) {
    const unsigned long long zero[kDbgSlots] = {};
    e = hipMemcpyToSymbol(HIP_SYMBOL(vrn_debug_counts), zero, sizeof(zero));
  }
  return e;
#else
  (void)out;
  (void)reset;
  return hipErrorNotSupported;
#endif
}

// ---------------------------------------------------------------------------
// scratch of the allocation-free render entry point (vrn_render_noalloc):
// the queue, blocks-done and statistics counters of one render, laid out as
// a workspace.  Every device the library runs on holds its own copy until
// the process ends.  Host code must never pass `scratch` itself to a kernel
// (in host code it is a stand-in, not a device address): it passes the
// address scratch_address() returns for the current device.
// ---------------------------------------------------------------------------
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

namespace {
std::mutex g_scratch_mu;
std::map<int, void*> g_scratch_ptr;   // device ordinal -> that device's copy of `scratch`
}  // namespace

hipError_t scratch_address(int device, void** out) {
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  auto it = g_scratch_ptr.find(device);
  if (it != g_scratch_ptr.end()) {
    *out = it->second;
    return hipSuccess;
  }
  // first call on this device (the caller made it current): take the
  // array's device address and clear the array once
  void* p = nullptr;
  hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  if (!p) return hipErrorInvalidSymbol;
  if ((e = launch_zero(p, kScratchBytes, nullptr)) != hipSuccess) return e;
  if ((e = hipStreamSynchronize(nullptr)) != hipSuccess) return e;
  g_scratch_ptr.emplace(device, p);
  *out = p;
  return hipSuccess;
}

hipError_t launch_zero(void* p, uint64_t bytes, hipStream_t s) {
  const uint64_t words = bytes / 4;
  const int grid = (int)std::min<uint64_t>((words + 255) / 256, 1024);
  hipLaunchKernelGGL(zero_kernel, dim3(std::max(grid, 1)), dim3(256), 0, s,
                     reinterpret_cast<uint32_t*>(p), words);
  return hipGetLastError();
}

hipError_t launch_rays(const vrn_camera* d_cams, uint32_t n_cams, uint32_t W, uint32_t H, float scale,
                       float* o, float* d, float* r, hipStream_t s) {
  const uint64_t n = (uint64_t)n_cams * W * H;
  hipLaunchKernelGGL(rays_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, d_cams, n_cams, W, H,
                     scale, o, d, r);
  return hipGetLastError();
}

hipError_t launch_march(const FieldDev& F, const vrn_camera* d_cams, uint32_t n_cams, uint32_t W,
                        uint32_t H, uint32_t* klist, uint32_t max_k, uint32_t* count, hipStream_t s) {
  const uint64_t n = (uint64_t)n_cams * W * H;
  if (F.lat)
    hipLaunchKernelGGL(march_kernel<1>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, F, d_cams, n_cams, W,
                       H, klist, max_k, count);
  else
    hipLaunchKernelGGL(march_kernel<0>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, F, d_cams, n_cams, W,
                       H, klist, max_k, count);
  return hipGetLastError();
}

hipError_t launch_encode(const FieldDev& F, const float* xyz, const float* t, const float* r, uint32_t n,
                         float* feat, hipStream_t s) {
  const uint64_t per_block = (kBlock / 64) * 16;
  const dim3 gr((unsigned)(((uint64_t)n + per_block - 1) / per_block)), bl(kBlock);
  if (F.table_f16) hipLaunchKernelGGL((encode_kernel<true>), gr, bl, 0, s, F, xyz, t, r, n, feat);
  else hipLaunchKernelGGL((encode_kernel<false>), gr, bl, 0, s, F, xyz, t, r, n, feat);
  return hipGetLastError();
}

template <int MODE>
static void launch_mlp_mode(const FieldDev& F, const float* feat, const float* dir, uint32_t n, float* sigma, float* rgb,
                            int n_cu, hipStream_t s) {
  static int per_cu = -1;
  if (per_cu < 0) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, mlp_kernel<MODE>, kMlpThreads, 0) != hipSuccess || nb < 1)
      nb = 1;
    per_cu = nb;
  }
  const MlpShape shape = mlp_shape(n, (uint32_t)n_cu, (uint32_t)per_cu);
  hipLaunchKernelGGL(mlp_kernel<MODE>, dim3(shape.grid), dim3(shape.threads), 0, s, F, feat, dir, n, sigma, rgb);
}

hipError_t launch_mlp(const FieldDev& F, const float* feat, const float* dir, uint32_t n, int compute,
                      float* sigma, float* rgb, int n_cu, hipStream_t s) {
  if (compute == 0) launch_mlp_mode<0>(F, feat, dir, n, sigma, rgb, n_cu, s);
  else if (compute == 1) launch_mlp_mode<1>(F, feat, dir, n, sigma, rgb, n_cu, s);
  else if (compute == 3) launch_mlp_mode<3>(F, feat, dir, n, sigma, rgb, n_cu, s);
  else launch_mlp_mode<2>(F, feat, dir, n, sigma, rgb, n_cu, s);
  return hipGetLastError();
}

}  // namespace vrn
