// Packed whole+shard attention forward in fp32, on the fp32 matrix cores.
//
// Same work items and outputs as the bf16 MFMA kernel; every product and sum
// is fp32 (v_mfma_f32_32x32x2_f32).  A workgroup of NW = 4 waves takes 32 query rows
// of an item, and wave w the 32-key blocks w, w+NW, ... of its keys:
//   S^T = K Q^T    one query per lane (Q in registers as the B operand), K
//                  straight from memory as A: a lane's 16-byte load of a key
//                  row feeds four MFMAs, which fixes the order in which d is
//                  summed (Q is held in the same order)
//   online softmax per query in the lane's registers
//   O^T += V^T P^T P's registers are the B operand as they stand (a register
//                  holds two keys, one in each half of the wave); V^T from
//                  16-byte loads of a value row, each feeding the four (two
//                  for d = 64) d blocks of the output
// No wave shares a key with another, so nothing is staged in LDS and the loop
// has no barrier; the partial results of a query are combined through
// LDS at the end.
//
// Bound: the fp32 matrix rate (4 d FLOP per pair), with 32 query rows so that
// a 1560-token image of 12 heads (588 tiles) fills the 256 CUs.  It replaces
// one query per lane on the vector ALUs, keys visited one by one (64 threads
// per workgroup, about one wave per CU for that image).  Measured there (d =
// 128, 15.0 GFLOP): 3,768 us before, 170 us now (88 TFLOP/s; a plain fp32
// library GEMM reaches 153), two workgroups per CU, which share a CU's matrix
// cores and so even out its last rounds; the error against fp64 was 1.0e-6 before
// and is 4.9e-7.  NW = 8 (one workgroup per CU) takes 186 us, and 50.7 instead of
// 52.7 us for 152 tiles; NW decides which keys a wave sums, so it is the same in every
// launch: a segment's bits do not depend on what else the launch holds.

#include "zl_device.h"
#include "zl_internal.h"

namespace zl {
namespace {

constexpr int BM = 32;               // query rows per workgroup
constexpr int BN = 32;               // keys per block
constexpr int NW = 4;                // waves per workgroup
constexpr int SUB = kFwd32TileM / BM;  // workgroups per work item
static_assert(kFwd32TileM % BM == 0 && kFwd32TileN == BN, "tile shapes");

__device__ __forceinline__ f32x16 mfma32f(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

template <int D>
__global__ __launch_bounds__(64 * NW, 2) void fwd_fp32_kernel(FwdParams p) {
  constexpr int NC = D / 8;    // 16-byte K loads per block and lane
  constexpr int DB = D / 32;   // output blocks of 32 d
  constexpr int PF = 8;        // loads in flight per wave
  __shared__ __attribute__((aligned(16))) f32x4 xo[NW][16 * DB / 4][64];
  __shared__ float xm[NW][64], xl[NW][64];

  const int n = p.n_items * SUB;
  for (int b = blockIdx.x; b < n; b += gridDim.x, __syncthreads()) {
    const int w = dispatch_item(b, n, p.xcd_chunk);
    Item it = p.items[w / SUB];
    const int sub = (w % SUB) * BM;
    if (sub >= it.q_len) continue;
    it.q_start += sub;
    it.q_len = min(it.q_len - sub, BM);

    const int lane = threadIdx.x & 63, ln = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t rs = (int64_t)p.num_heads * D;
    const uint32_t row_bytes = (uint32_t)rs * 4u;
    const float* kg = static_cast<const float*>(p.k) + ((int64_t)it.k_start * p.num_heads + it.head) * D;
    const float* vg = static_cast<const float*>(p.v) + ((int64_t)it.k_start * p.num_heads + it.head) * D;
    const int64_t row = (int64_t)(it.q_start + ln) * p.num_heads + it.head;
    const bool q_ok = ln < it.q_len;

    // Q in the order of the S MFMAs: MFMA 4c+j multiplies d = 8c + 4g + j.
    f32x4 q[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
      q[c] = q_ok ? *reinterpret_cast<const f32x4*>(static_cast<const float*>(p.q) + row * D + 8 * c + 4 * g)
                  : f32x4{0.f, 0.f, 0.f, 0.f};

    // o[db][i]: d = DB*m + db with m = 8*(i/4) + 4g + i%4, query ln.
    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = f32x16{};
    float m = -INFINITY, l = 0.f;

    // The wave's loads run as one stream, PF ahead: a block's NC loads of K, its
    // 16 of V, then the next block's.  Rows past the range (and whole blocks past
    // it) read zero through the range check of the block's buffer resource.
    struct Ring { f32x4 v[PF]; } ring;
    const uint32_t koff = (uint32_t)ln * row_bytes + 16u * g;
    uint32_t voff = 4u * g * row_bytes + (uint32_t)ln * (4u * DB);
    auto rsrc_of = [&](const float* base, int kt) __attribute__((always_inline)) {
      const int nv = min(it.k_len - kt, BN);
      const uint32_t bytes = nv > 0 ? (uint32_t)(nv - 1) * row_bytes + D * 4u : 0u;
      const float* at = base + (int64_t)(nv > 0 ? kt : 0) * rs;
      return __builtin_amdgcn_make_buffer_rsrc((void*)at, 0, bytes, 0x00020000);
    };
    auto load_k = [&](__amdgpu_buffer_rsrc_t r, int c) __attribute__((always_inline)) {
      return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, koff + 32u * c, 0, 0));
    };
    // V of P register i: keys 8*(i/4) + i%4 and 4 more, d = DB*ln ...
    auto load_v = [&](__amdgpu_buffer_rsrc_t r, int i) __attribute__((always_inline)) {
      const uint32_t at = voff + (uint32_t)(8 * (i >> 2) + (i & 3)) * row_bytes;
      if constexpr (DB == 4) {
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, at, 0, 0));
      } else {
        const f32x2 x = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(r, at, 0, 0));
        return f32x4{x[0], x[1], 0.f, 0.f};
      }
    };

    constexpr int NL = NC + 16;  // loads per block; a multiple of PF, so that ring slots are literals
    static_assert(NL % PF == 0 && NC >= PF, "load ring");
    int kt = wave * BN;
    {
      const auto kr = rsrc_of(kg, kt);
#pragma unroll
      for (int c = 0; c < PF; ++c) ring.v[c] = load_k(kr, c);
    }
    for (; kt < it.k_len; kt += NW * BN) {
      const auto kr = rsrc_of(kg, kt), vr = rsrc_of(vg, kt), kn = rsrc_of(kg, kt + NW * BN);
      auto advance = [&](int j) __attribute__((always_inline)) {  // load j + PF of the stream into slot j % PF
        const int n = j + PF;
        if (n < NC) ring.v[j % PF] = load_k(kr, n);
        else if (n < NL) ring.v[j % PF] = load_v(vr, n - NC);
        else ring.v[j % PF] = load_k(kn, n - NL);
      };
      asm volatile("" : "+v"(voff));  // keeps the 16 V row offsets from being held across blocks
      f32x16 s = f32x16{};
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const f32x4 a = ring.v[c % PF];
        advance(c);
#pragma unroll
        for (int j = 0; j < 4; ++j) s = mfma32f(a[j], q[c][j], s);
        __builtin_amdgcn_sched_barrier(0);
      }
      // s[i]: key 8*(i/4) + 4g + i%4 of the block, query ln.
      const int nvalid = it.k_len - kt;
      float mb = -INFINITY;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s[i] = (8 * (i >> 2) + 4 * g + (i & 3)) < nvalid ? s[i] * p.scale : -INFINITY;
        mb = fmaxf(mb, s[i]);
      }
      const float m_new = fmaxf(m, xor32_max(mb));
      const float ref = m_new == -INFINITY ? 0.f : m_new;  // every score so far is -inf
      const float alpha = expf(m - ref);
      m = m_new;
      float ls = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s[i] = expf(s[i] - ref);
        ls += s[i];
      }
      l = l * alpha + ls;
      if (__any(alpha != 1.f)) {
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db] *= alpha;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const f32x4 a = ring.v[(NC + i) % PF];
        advance(NC + i);
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db] = mfma32f(a[db], s[i], o[db]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }

    // Combine the waves: slot 16-byte group t of a lane holds o values of DB
    // consecutive d per i (t = i for d = 128; two i for d = 64).
    constexpr int GROUPS = 16 * DB / 4;
#pragma unroll
    for (int t = 0; t < GROUPS; ++t) {
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = o[e % DB][t * 4 / DB + e / DB];
      xo[wave][t][lane] = x;
    }
    xm[wave][lane] = m;
    xl[wave][lane] = xor32_sum(l);
    // Every wave reads the running statistic before the barrier, wave 0 replaces
    // it after.
    const bool step = it.slot >= 0 && p.step_mode;
    const float lse_prev = step && !p.step_first && q_ok ? p.lse_acc[row] : 0.f;
    __syncthreads();
    float mt = xm[0][lane];
#pragma unroll
    for (int v = 1; v < NW; ++v) mt = fmaxf(mt, xm[v][lane]);
    const float ref = mt == -INFINITY ? 0.f : mt;
    float lt = 0.f, wgt[NW];
#pragma unroll
    for (int v = 0; v < NW; ++v) {
      wgt[v] = expf(xm[v][lane] - ref);
      lt += wgt[v] * xl[v][lane];
    }
    const float inv = lt > 0.f ? 1.f / lt : 0.f;
    const float lse = lt > 0.f ? mt + logf(lt) : -INFINITY;
    // Ring step: fold this block into the running accumulator (see the bf16 kernel).
    float wa = 0.f, wb = 1.f, lse_out = lse;
    if (step) step_weights(p.step_first, lse_prev, lse, wa, wb, lse_out);
    wb *= inv;
    float* og = static_cast<float*>(p.out) + row * D;
    if (it.slot >= 0) {
      if (!step) og = static_cast<float*>(p.o_part) + it.slot * p.slot_stride + row * D;
      else if (!p.step_last) og = p.o_acc + row * D;
    }
    // Wave w writes groups w*GROUPS/NW ...; d0 is the group's first d.
#pragma unroll
    for (int e = 0; e < GROUPS / NW; ++e) {
      const int t = wave * (GROUPS / NW) + e;
      f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < NW; ++v) x += wgt[v] * xo[v][t][lane];
      const int i = t * 4 / DB;
      const int d0 = DB * (8 * (i >> 2) + 4 * g + (i & 3));
      if (!q_ok) continue;
      if (step) {
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
        if (!p.step_first) a = *reinterpret_cast<const f32x4*>(p.o_acc + row * D + d0);
        x = wa * a + wb * x;
      } else {
        x *= inv;
      }
      *reinterpret_cast<f32x4*>(og + d0) = x;
    }
    if (wave != 0 || g != 0 || !q_ok) continue;
    if (it.slot < 0) p.lse[row] = lse;
    else if (!step) p.lse_part[it.slot * p.lse_slot_stride + row] = lse;
    else (p.step_last ? p.lse : p.lse_acc)[row] = lse_out;
  }
}

template <int D>
hipError_t launch_d(const FwdParams& p, hipStream_t s) {
  // The grid's thread count has to stay below 2^32: further tiles are taken in turn.
  const int64_t tiles = (int64_t)p.n_items * SUB;
  const dim3 grid((unsigned)(tiles < (1 << 20) ? tiles : (1 << 20)));
  hipLaunchKernelGGL(fwd_fp32_kernel<D>, grid, dim3(64 * NW), 0, s, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd_fp32(const FwdParams& p, int head_dim, hipStream_t s) {
  return head_dim == 128 ? launch_d<128>(p, s) : launch_d<64>(p, s);
}

}  // namespace zl
