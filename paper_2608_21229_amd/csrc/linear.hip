// Dense bf16 projection for the chained synthetic layer: out = A W^T (+ R).
//
// The layer around the attention (Sec. 3.1, Eq. 2: K_R = R W_K, V_R = R W_V
// per layer; the output projection and residual feed the next layer) is a
// plain GEMM per token: out[m, n] = sum_k A[m, k] W[n, k] (+ R[m, n]), fp32
// accumulation, one bf16 rounding (RNE) at the end.
//
// Output tiles of 256 x 256 down to 64 x 64 (one work-group each, chosen by
// the number of rounds over the CUs; a partial last round of 256 x 256 tiles
// may run in smaller ones); each wave owns a block of
// v_mfma_f32_32x32x16_bf16 accumulators.  K advances in slices of 64: the A
// and W tiles (64 k per row, 128-byte rows) stream through an LDS ring with
// direct global->LDS loads; 16-byte granule g of row r is stored at slot
// g ^ ((r >> 1) & 7), so the 128-bit fragment reads of 16 consecutive rows hit
// 16 distinct bank groups.  Every output element is one chain of MFMAs over
// k in steps of 16, in the same order in every tile, so a row's result depends
// neither on the other rows nor on the tile that holds it.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rc_internal.h"

namespace rc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kLinBK = 64;  // k per 128-byte LDS row

__device__ __forceinline__ uint32_t lds_u32(const char* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const lds_void*)p));
}

// 16 bytes per lane straight into LDS at M0 + 16 lane; offsets past the
// record count read as zeros (see the attention kernel for the wait rules).
__device__ __forceinline__ void dma16(uint32_t lds, uint32_t voff, __amdgpu_buffer_rsrc_t rsrc) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(lds), "v"(voff), "s"(rsrc)
               : "memory", "m0");
}

__device__ __forceinline__ int lin_swz(int row, int g) { return g ^ ((row >> 1) & 7); }

// A tile of 64 k per row is loaded in 1 KB chunks of 8 rows; lane l of chunk c
// fills LDS slot p = 64 c + l: row p / 8, slot p % 8, holding the row's granule
// slot ^ ((row >> 1) & 7).  `ld` is the row stride in elements.
__device__ __forceinline__ uint32_t lin_off(int chunk, int lane, int64_t ld) {
  const int p = chunk * 64 + lane;
  const int row = p >> 3, slot = p & 7;
  return uint32_t(row) * uint32_t(ld) * 2u + uint32_t(lin_swz(row, slot)) * 16u;
}

// 128-bit fragment of rows r0 + lane % 32, k = 16 kk + 8 (lane / 32) .. +7.
__device__ __forceinline__ bf16x8 lin_frag(const char* t, int r0, int lane, int kk) {
  const int row = r0 + (lane & 31);
  const int g = 2 * kk + (lane >> 5);
  return *reinterpret_cast<const bf16x8*>(t + row * (kLinBK * 2) + lin_swz(row, g) * 16);
}

__device__ __forceinline__ void lin_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
}

// Scheduling fence: the compiler moves no instruction across it.
__device__ __forceinline__ void lin_fence() { __builtin_amdgcn_sched_barrier(0); }

// The hardware deals work-groups round-robin to the 8 XCDs; give each XCD a
// contiguous run of logical tiles.
__device__ __forceinline__ int64_t lin_xcd_block(int64_t bid, int64_t nblk) {
  const int64_t xcd = bid & 7, kx = bid >> 3, per = nblk >> 3, rem = nblk & 7;
  return (xcd < rem) ? xcd * (per + 1) + kx : rem * (per + 1) + (xcd - rem) * per + kx;
}

// Logical tile of this work-group: groups of kGroupM m-tiles, m fastest inside
// a group, so that the work-groups an XCD runs together share A and W tiles.
constexpr int kGroupM = 4;
template <int BM, int BN>
__device__ __forceinline__ void lin_tile(const LinearParams& q, int64_t w, int64_t& m0, int& n0) {
  const int64_t n_tiles = q.N / BN;
  const int64_t m_tiles = (q.M + BM - 1) / BM;
  const int64_t per_group = int64_t(kGroupM) * n_tiles;
  const int64_t first_m = (w / per_group) * kGroupM;
  const int64_t group_m = min(int64_t(kGroupM), m_tiles - first_m);
  const int64_t in_group = w % per_group;
  m0 = (first_m + in_group % group_m) * BM;
  n0 = int(in_group / group_m) * BN;
}

// One 32 x 32 accumulator block (row m of A, columns n .. n + 31) to out: the
// lane of half hh holds columns 8 (r / 4) + 4 hh + r % 4 of its row.  The two
// halves trade accumulators (slots 8 t + 4 .. +7 of the low half against slots
// 8 t .. +3 of the high half), so that a lane owns eight consecutive columns
// and reads and writes 16 bytes.
__device__ __forceinline__ void lin_store_block(const LinearParams& q, f32x16 acc, int64_t m, int n, int hh) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[8 * t + j]),
                                                      __float_as_uint(acc[8 * t + 4 + j]), false, false);
      v[j] = __uint_as_float(s[0]);
      v[4 + j] = __uint_as_float(s[1]);
    }
    if (m < q.M) {
      const int64_t c = n + 16 * t + 8 * hh;
      if (q.r) {
        const bf16x8 rb = *reinterpret_cast<const bf16x8*>(q.r + m * q.ldr + c);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += float(rb[e]);
      }
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (__bf16)v[e];
      *reinterpret_cast<bf16x8*>(q.out + m * q.ldo + c) = o;
    }
  }
}

// One BM x BN output tile: WM x WN waves, each MB x NB accumulators of 32 x 32.
// A ring of ST stages, each KS slices of the A and W tile; ST - 1 stages are
// in flight while one is computed.  Slices past K load zeros (record count 0),
// so every step issues the same loads.
//
// What bounds it: the loads (64 KB a slice for 256 x 256) and the fragment
// reads share the LDS, whose 2 048 cycles a slice equal the MFMAs' there.  A
// burst of loads at the start of a step keeps every wave from its MFMAs (about
// 500 cycles a step whatever the tile), so they go out one at a time between
// the MFMAs of the step's first SP / 8: in all of it where several stages are
// in flight, in the first 3/8 with two stages, whose loads must land by the
// step's end (1/8, 1/4, 3/8, 1/2, 3/4: 1.12, 1.10, 1.09, 1.15, 1.17 ms at
// 25 152 x 9216 x 3072; one burst 1.18 ms.  256 x 128 at 1536 x 3072 x 3072:
// 39 us -> 34 us).  Measured and not kept: the next step's first fragments read
// before the barrier, 128 x 128 blocks on four waves (within noise), 128 x 256
// tiles, 32-row tiles, two work-groups per CU for the small tiles.
template <int MB, int NB, int WM, int WN, int KS, int ST, int SP>
__device__ __forceinline__ void linear_tile(const LinearParams& q, char* ring, int64_t m0, int n0) {
  constexpr int NW = WM * WN;
  constexpr int BM = 32 * MB * WM, BN = 32 * NB * WN;
  constexpr int CA = BM / 8 / NW, CW = BN / 8 / NW;  // 1 KB chunks per wave per slice
  static_assert(CA * NW * 8 == BM && CW * NW * 8 == BN, "chunks divide over the waves");
  constexpr int kSlice = (BM + BN) * kLinBK * 2, kStage = KS * kSlice;
  constexpr int kLoads = KS * (CA + CW);
  static_assert(ST * kLoads <= 63, "vmcnt range");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;

  uint32_t aoff[CA], woff[CW];
#pragma unroll
  for (int i = 0; i < CA; ++i) aoff[i] = lin_off(i * NW + wave, lane, q.lda);
#pragma unroll
  for (int i = 0; i < CW; ++i) woff[i] = lin_off(i * NW + wave, lane, q.K);
  const int a_rows = int(min(int64_t(BM), q.M - m0));
  const int nrec_a = int(int64_t(a_rows - 1) * q.lda * 2 + kLinBK * 2);  // rows past M load zeros
  const int nrec_w = int(int64_t(BN - 1) * q.K * 2 + kLinBK * 2);
  const uint16_t* pa = q.a + m0 * q.lda;
  const uint16_t* pw = q.w + int64_t(n0) * q.K;
  const uint32_t lds0 = lds_u32(ring) + uint32_t(wave) * 1024u;

  // load l of this wave for the stage of slices slice0 .. slice0 + KS - 1
  const auto issue1 = [&](int slice0, uint32_t stage, int l) {
    const int s = l / (CA + CW), i = l % (CA + CW);
    const int k0 = (slice0 + s) * kLinBK;
    const bool in = k0 < q.K;
    const int kc = in ? k0 : 0;
    const uint32_t base = lds0 + stage + uint32_t(s * kSlice);
    if (i < CA) {
      const __amdgpu_buffer_rsrc_t ra =
          __builtin_amdgcn_make_buffer_rsrc((void*)(pa + kc), (short)0, in ? nrec_a : 0, 0x00020000);
      dma16(base + uint32_t(i * NW * 1024), aoff[i], ra);
    } else {
      const __amdgpu_buffer_rsrc_t rw =
          __builtin_amdgcn_make_buffer_rsrc((void*)(pw + kc), (short)0, in ? nrec_w : 0, 0x00020000);
      dma16(base + uint32_t(BM * kLinBK * 2 + (i - CA) * NW * 1024), woff[i - CA], rw);
    }
  };
  const auto issue = [&](int slice0, uint32_t stage) {
#pragma unroll
    for (int l = 0; l < kLoads; ++l) issue1(slice0, stage, l);
  };

  f32x16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  constexpr int NF = MB + NB, NM = MB * NB, NC = KS * (kLinBK / 16);
  // fragments are read PF chunks ahead of their MFMAs
  constexpr int PF = NM >= 4 ? 1 : NM >= 2 ? 2 : 4;
  bf16x8 fr[PF + 1][NF];
  // fragment t of 16-wide k chunk c: A rows for t < MB, W rows otherwise
  const auto frag = [&](const char* st, int c, int t) {
    const char* sl = st + (c / 4) * kSlice;
    return t < MB ? lin_frag(sl, wm * 32 * MB + t * 32, lane, c % 4)
                  : lin_frag(sl + BM * kLinBK * 2, wn * 32 * NB + (t - MB) * 32, lane, c % 4);
  };
  const int steps = (q.K / kLinBK + KS - 1) / KS;
#pragma unroll
  for (int s = 0; s < ST - 1; ++s) issue(s * KS, uint32_t(s * kStage));
  uint32_t cur = 0, fill = (ST - 1) * kStage;
  for (int s = 0; s < steps; ++s) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((ST - 2) * kLoads) : "memory");
    lin_barrier();
    const char* st = ring + cur;
#pragma unroll
    for (int c = 0; c < PF; ++c)
#pragma unroll
      for (int t = 0; t < NF; ++t) fr[c][t] = frag(st, c, t);
    lin_fence();
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int t = 0; t < (NM > NF ? NM : NF); ++t) {
        if (t < NM) {
          const int i = t / NB, j = t % NB;
          // C^T block (n rows, m columns): the accumulator holds one output
          // row m per lane (lane % 32)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[c % (PF + 1)][MB + j], fr[c % (PF + 1)][i],
                                                              acc[i][j], 0, 0, 0);
        }
        if (c + PF < NC && t < NF) fr[(c + PF) % (PF + 1)][t] = frag(st, c + PF, t);
        if (t < NM) {
#pragma unroll
          for (int l = 0; l < kLoads; ++l)
            if (l * (NC * NM * SP / 8) / kLoads == c * NM + t) issue1((s + ST - 1) * KS, fill, l);
        }
        lin_fence();
      }
    }
    cur = cur + kStage == ST * kStage ? 0 : cur + kStage;
    fill = fill + kStage == ST * kStage ? 0 : fill + kStage;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load into LDS outlives the work-group

#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
      lin_store_block(q, acc[i][j], m0 + wm * 32 * MB + i * 32 + (lane & 31), n0 + wn * 32 * NB + j * 32, lane >> 5);
}

template <int MB, int NB, int WM, int WN, int KS, int ST>
constexpr int kRingBytes = ST * KS * 32 * (MB * WM + NB * WN) * kLinBK * 2;

// A grid of one tile size.
template <int MB, int NB, int WM, int WN, int KS, int ST, int SP>
__global__ __launch_bounds__(WM * WN * 64) void linear_kernel(const LinearParams q) {
  __shared__ __attribute__((aligned(1024))) char ring[kRingBytes<MB, NB, WM, WN, KS, ST>];
  int64_t m0;
  int n0;
  lin_tile<32 * MB * WM, 32 * NB * WN>(q, lin_xcd_block(blockIdx.x, gridDim.x), m0, n0);
  linear_tile<MB, NB, WM, WN, KS, ST, SP>(q, ring, m0, n0);
}

// A grid of 256 x 256 tiles whose last partial round is cut into smaller parts,
// so that the round ends sooner: tiles from `whole` on (logical order) run in
// parts of kLinPartM[part] x 128, on the CUs that become free.  Same bits
// as whole tiles.  A round of whole tiles takes 77 us at K = 3072 in a grid of
// four (MFMAs in 71% of the cycles, at 1.74 GHz; in one round 62%, at 1.91
// GHz): the clock falls as more CUs work, so cutting only recovers what a
// round's idle CUs do not give back in clock: 1.125 rounds of N = 9216, K = 3072
// 117 -> 96 us, 2.1 rounds 207 -> 178, 2.25 rounds 212 -> 185, 4.2 rounds 361 ->
// 336; 1.1 rounds of N = K = 1024 49 -> 40 us.  The two smaller parts run on
// four of the work-group's waves: as fast as on eight.
__global__ __launch_bounds__(512) void linear_cut_kernel(const LinearParams q, const LinearPlan cut) {
  __shared__ __attribute__((aligned(1024))) char ring[kRingBytes<2, 2, 4, 2, 1, 3>];
  static_assert(sizeof(ring) >= size_t(kRingBytes<4, 2, 2, 4, 1, 2>), "ring");
  static_assert(sizeof(ring) >= size_t(kRingBytes<2, 2, 2, 2, 1, 4>), "ring");
  static_assert(sizeof(ring) >= size_t(kRingBytes<2, 1, 1, 4, 1, 6>), "ring");
  int64_t m0;
  int n0;
  if (int64_t(blockIdx.x) < cut.whole) {
    lin_tile<256, 256>(q, lin_xcd_block(blockIdx.x, cut.whole), m0, n0);
    linear_tile<4, 2, 2, 4, 1, 2, 3>(q, ring, m0, n0);
    return;
  }
  const int parts = lin_parts(cut.part);
  const int64_t w = lin_xcd_block(blockIdx.x - cut.whole, (cut.tiles - cut.whole) * parts);
  lin_tile<256, 256>(q, cut.whole + w / parts, m0, n0);
  m0 += int(w % parts) / 2 * kLinPartM[cut.part];
  n0 += int(w % parts) % 2 * 128;
  if (m0 >= q.M) return;
  if (cut.part < 2 && threadIdx.x >= 256) return;  // barriers wait for the waves that remain
  switch (cut.part) {
    case 0: linear_tile<2, 1, 1, 4, 1, 6, 3>(q, ring, m0, n0); break;
    case 1: linear_tile<2, 2, 2, 2, 1, 4, 8>(q, ring, m0, n0); break;
    default: linear_tile<2, 2, 4, 2, 1, 3, 8>(q, ring, m0, n0); break;
  }
}

template <int MB, int NB, int WM, int WN, int KS, int ST, int SP>
void launch_tile(const LinearParams& q, hipStream_t s) {
  constexpr int BM = 32 * MB * WM, BN = 32 * NB * WN;
  const int64_t blocks = ((q.M + BM - 1) / BM) * (q.N / BN);
  hipLaunchKernelGGL((linear_kernel<MB, NB, WM, WN, KS, ST, SP>), dim3(blocks), dim3(WM * WN * 64), 0, s, q);
}

}  // namespace

int launch_linear(const LinearParams& q, void* stream) {
  if (q.M == 0) return 0;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const LinearPlan plan = plan_linear(q);
  if (plan.part >= 0) {
    const int64_t blocks = plan.whole + (plan.tiles - plan.whole) * lin_parts(plan.part);
    hipLaunchKernelGGL(linear_cut_kernel, dim3(blocks), dim3(512), 0, s, q, plan);
    return int(hipGetLastError());
  }
  switch (plan.tile) {
    case 0: launch_tile<4, 2, 2, 4, 1, 2, 3>(q, s); break;
    case 1: launch_tile<2, 2, 4, 2, 1, 3, 8>(q, s); break;
    case 2: launch_tile<2, 2, 2, 2, 1, 4, 8>(q, s); break;
    case 3: launch_tile<2, 1, 1, 4, 1, 6, 3>(q, s); break;
    default: launch_tile<1, 1, 2, 2, 2, 4, 2>(q, s); break;
  }
  return int(hipGetLastError());
}

}  // namespace rc
