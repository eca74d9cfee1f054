// fp32 split-KV decode on the matrix cores (v_mfma_f32_16x16x4_f32, fp32 products and sums).
//
// As in the bf16 kernel a workgroup streams one chunk of one participant's cache segment for one
// KV head against all query columns that may see it, 16 NQ columns per workgroup.  The 4 wavefronts
// take 16 rows each of every 64-row tile; S^T = K Q^T leaves the scores of one column in one lane
// group, where they are the B operand of O^T += V^T P^T as they stand (layouts as in prefill_f32.hip).
// A 64-row tile costs a CU 16 D NQ matrix cycles and 512 D bytes of loads, so up to 64 columns the
// chip is bound by memory, and short caches by the launches: 5 participants with 200..1500 rows,
// 8/2 heads of 64, one local and one sync block (6 MB): 17.7 us, where one wavefront per (participant, head)
// took 1525 us.
#include <math.h>

#include "common.h"
#include "decode_walk.h"
#include "mfma_tile.h"

namespace fedattn {

namespace {

// tiles in flight or in use: two K/V tile pairs up to 128 columns (one streams in while the other is
// worked on), one beyond that
template <int DP>
constexpr int f32_stages() { return DP > 128 ? 1 : 2; }
template <int DP>
constexpr int f32_smem_bytes() { return f32_stages<DP>() * 2 * kKvTile * DP * 4; }

template <int DP, int NQ, bool PIECES>
__global__ __launch_bounds__(256, 1) void decode_f32_kernel(DecodeArgs a) {
  constexpr int CH = DP / 4;               // 16-byte chunks per row
  constexpr int ROWB = DP * 4;
  constexpr int TILEB = kKvTile * ROWB;
  constexpr int IPW = TILEB / 1024 / 4;    // direct-to-LDS loads per wavefront and tile
  constexpr int DS = DP / 16;
  constexpr int STAGES = f32_stages<DP>();
  static_assert(4 * NQ * DS * 1024 <= f32_smem_bytes<DP>(), "the merge reuses the tile stages");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];  // stage s: K tile, V tile
  __shared__ float ml_s[4][NQ][2][16];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kg = lane >> 4;
  const lds_cptr lds0 = (lds_cptr)(lds_void_ptr)smem;
  const uint32_t lds_base = lds_addr_of(smem);

  const int bz = blockIdx.z;               // block of a fused launch
  const int64_t blk = a.block_list[bz];
  const float* q_ptr = reinterpret_cast<const float*>(reinterpret_cast<const unsigned char*>(a.q) + blk * a.q_block_bytes);
  float* out_ptr = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(a.out) + blk * a.q_block_bytes);
  float* part_o = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(a.part_o) + bz * a.slice_bytes);
  float* part_ml = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(a.part_ml) + bz * a.slice_bytes);
  uint64_t* counters = reinterpret_cast<uint64_t*>(reinterpret_cast<unsigned char*>(a.counters) + bz * a.slice_bytes);

  const int Hq = a.Hq, Hkv = a.Hkv, D = a.D;
  const int G = Hq / Hkv;
  const DecodePiece pc = decode_piece<PIECES>(a);
  const int g = pc.g0 + blockIdx.x % pc.n_g;
  const int gc = blockIdx.x / pc.n_g;
  const int col0 = pc.col0 + blockIdx.y * 16 * NQ, col_end = pc.col0 + pc.n_cols;
  const DecodeChunk ch = find_decode_chunk(a, gc, lane);
  const int m = ch.m;
  const int nt = (ch.r_hi - ch.r_lo + kKvTile - 1) / kKvTile;
  const int row_elems = Hkv * D;
  const int64_t first = ((int64_t)(ch.seg_row0 + ch.r_lo) * Hkv + g) * D;
  const float* k_ptr = reinterpret_cast<const float*>(reinterpret_cast<const unsigned char*>(a.k_cache) + blk * a.cache_block_bytes);
  const float* v_ptr = reinterpret_cast<const float*>(reinterpret_cast<const unsigned char*>(a.v_cache) + blk * a.cache_block_bytes);
  const float *kbase = k_ptr + first, *vbase = v_ptr + first;

  // slot (row, cp) of a tile receives chunk cp ^ (row mod 8)
  auto issue = [&](int t) __attribute__((always_inline)) {
    const int len = min(kKvTile, ch.r_hi - ch.r_lo - kKvTile * t);
    const uint32_t stage = lds_base + (t % STAGES) * 2 * TILEB;
#pragma unroll
    for (int kv = 0; kv < 2; ++kv) {
      const float* base = (kv ? vbase : kbase) + (int64_t)t * kKvTile * row_elems;
#pragma unroll
      for (int i = 0; i < IPW; ++i) {
        const int sidx = (wave * IPW + i) * 64 + lane;
        const int row = sidx / CH, chunk = min((sidx % CH) ^ (row & 7), D / 4 - 1);
        lds_dma_16(base, (uint32_t)(min(row, len - 1) * row_elems + chunk * 4) * 4u, stage + kv * TILEB + (wave * IPW + i) * 1024);
      }
    }
  };

  // this lane's query columns (local block: head inside the KV group; sync block: participant * G + head)
  f32x4 q[NQ][DS];
  int limit[NQ];   // visible rows of this segment
#pragma unroll
  for (int iq = 0; iq < NQ; ++iq) {
    const int col = col0 + 16 * iq + l16;
    const bool ok = col < col_end;
    const int part = ok ? (a.is_sync ? col / G : m) : 0;
    const int head = ok ? g * G + (a.is_sync ? col % G : col) : 0;
    limit[iq] = ok ? (part == m ? ch.own_len : ch.rem_len) : 0;
    const float* qrow = q_ptr + ((int64_t)part * Hq + head) * D + 4 * kg;
#pragma unroll
    for (int s = 0; s < DS; ++s)
      q[iq][s] = 16 * s + 4 * kg < D ? *reinterpret_cast<const f32x4*>(qrow + 16 * s) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  issue(0);
  const MergeSet ms = merge_set(a, ch, g, counters);
  const bool set_up = NQ == 1 && a.merge_in_kernel && ms.count > 1 && a.ticket != 0;
  uint64_t cnt_found = 0;
  if (set_up) cnt_found = __hip_atomic_load(ms.cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  const int k_addr = (16 * wave + l16) * ROWB;
  const int k_swz = l16 & 7;
  int v_addr[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v_addr[e] = TILEB + (16 * wave + 4 * kg + e) * ROWB + (((l16 >> 2) ^ e) << 4) + (l16 & 3) * 4;
  const int v_half = (kg & 1) * 64;

  f32x4 o[NQ][DS];
  float m_run[NQ], l_run[NQ];
#pragma unroll
  for (int iq = 0; iq < NQ; ++iq) {
    m_run[iq] = -INFINITY;
    l_run[iq] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DS; ++dt) o[iq][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float sc = a.scale * kLog2e;

  for (int t = 0; t < nt; ++t) {
    if (STAGES == 1 && t > 0) {
      __syncthreads();   // everyone is done with the stage's last tile
      issue(t);
    }
    wait_vmcnt<0>();
    __syncthreads();     // tile t is complete in LDS, and everyone is done with tile t - 1
    if (STAGES > 1 && t + 1 < nt) issue(t + 1);
    const int st_off = (t % STAGES) * 2 * TILEB;
    const int row0 = ch.r_lo + kKvTile * t + 16 * wave;   // this wavefront's first cache row
    if (row0 >= ch.r_hi) continue;
    f32x4 s[NQ];
#pragma unroll
    for (int iq = 0; iq < NQ; ++iq) s[iq] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < DS; ++st) {
      const f32x4 kf = *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(
          lds0 + (st_off + k_addr + (((4 * st + kg) ^ k_swz) << 4)));
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int iq = 0; iq < NQ; ++iq) s[iq] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[e], q[iq][st][e], s[iq], 0, 0, 0);
    }
    if (row0 + 16 > ch.min_limit) {
#pragma unroll
      for (int iq = 0; iq < NQ; ++iq)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (row0 + 4 * kg + e >= limit[iq]) s[iq][e] = -INFINITY;
    }
#pragma unroll
    for (int iq = 0; iq < NQ; ++iq) {
      const float m_cand = max_over_kgroups(fmaxf(fmaxf(s[iq][0], s[iq][1]), fmaxf(s[iq][2], s[iq][3]))) * sc;
      if (__builtin_amdgcn_ballot_w64(m_cand > m_run[iq] + kRescaleThreshold) != 0) {
        const float m_new = fmaxf(m_run[iq], m_cand);
        const float alpha = __builtin_amdgcn_exp2f(m_run[iq] - ((m_new == -INFINITY) ? 0.f : m_new));
        m_run[iq] = m_new;
        l_run[iq] *= alpha;
#pragma unroll
        for (int dt = 0; dt < DS; ++dt) o[iq][dt] *= alpha;
      }
      const float m_use = (m_run[iq] == -INFINITY) ? 0.f : m_run[iq];
#pragma unroll
      for (int e = 0; e < 4; ++e) s[iq][e] = __builtin_amdgcn_exp2f(fmaf(s[iq][e], sc, -m_use));
      l_run[iq] += (s[iq][0] + s[iq][1]) + (s[iq][2] + s[iq][3]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int dt = 0; dt < DS; ++dt) {
        const float vf = *reinterpret_cast<const __attribute__((address_space(3))) float*>(
            lds0 + (st_off + v_addr[e] + (dt >> 1) * 128 + ((dt & 1) ? 64 - v_half : v_half)));
#pragma unroll
        for (int iq = 0; iq < NQ; ++iq) o[iq][dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf, s[iq][e], o[iq][dt], 0, 0, 0);
      }
  }

  if (set_up) claim_counter(ms, cnt_found, a.ticket);
  // merge the 4 wavefronts through LDS, each taking every fourth slice of the head dimension
  __shared__ uint32_t odd_s;   // output columns that came out not finite
  if (tid == 0) odd_s = 0;
  __syncthreads();
  f32x4* xo = reinterpret_cast<f32x4*>(smem) + lane;
#pragma unroll
  for (int iq = 0; iq < NQ; ++iq) {
    l_run[iq] = sum_over_kgroups(l_run[iq]);
    if (kg == 0) {
      ml_s[wave][iq][0][l16] = m_run[iq];
      ml_s[wave][iq][1][l16] = l_run[iq];
    }
#pragma unroll
    for (int dt = 0; dt < DS; ++dt) xo[((wave * NQ + iq) * DS + dt) * 64] = o[iq][dt];
  }
  __syncthreads();
#pragma unroll
  for (int iq = 0; iq < NQ; ++iq) {
    const int col = col0 + 16 * iq + l16;
    if (col >= col_end) continue;
    float mm = -INFINITY, den = 0.f, f[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) mm = fmaxf(mm, ml_s[k][iq][0][l16]);
    const float mu = (mm == -INFINITY) ? 0.f : mm;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      f[k] = __builtin_amdgcn_exp2f(ml_s[k][iq][0][l16] - mu);
      den = fmaf(ml_s[k][iq][1][l16], f[k], den);
    }
    const int64_t prow = partial_row(a, pc, g, gc, col);
    const bool only = a.merge_in_kernel && ms.count == 1;   // nothing to merge: the output row itself
    const float norm = only ? (den > 0.f ? 1.f / den : 0.f) : 1.f;
    float* dst = only ? out_ptr + decode_out_row(a, g, m, col) * D : part_o + prow * D;
    for (int dt = wave; dt < DS; dt += 4) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < 4; ++k) acc += xo[((k * NQ + iq) * DS + dt) * 64] * f[k];
      acc *= norm;
      if (16 * dt + 4 * kg >= D) continue;
      if (NQ > 1 || only) {
        *reinterpret_cast<f32x4*>(dst + 16 * dt + 4 * kg) = acc;
        if (NQ == 1) note_nonfinite(acc, l16, &odd_s);
      } else {
        store_pair_agent(dst + 16 * dt + 4 * kg, acc[0], acc[1]);
        store_pair_agent(dst + 16 * dt + 4 * kg + 2, acc[2], acc[3]);
      }
    }
    if (!only && wave == 0 && kg == 0) store_pair_agent(part_ml + prow * 2, mm, den);
  }
  if (NQ == 1 && a.merge_in_kernel) {
    if (ms.count > 1) {
      merge_if_last<float, true>(a, ms, g, m, D, part_o, part_ml, out_ptr, q_ptr, k_ptr, v_ptr);
    } else {
      lds_barrier();
      if (__builtin_expect(odd_s != 0, 0)) redo_decode_columns<float, 4>(q_ptr, k_ptr, v_ptr, out_ptr, g, m, 0, odd_s);
    }
  }
}

template <int DP, int NQ, bool PIECES = false>
hipError_t launch_decode_f32_t(const DecodeArgs& a, int n_z, hipStream_t s) {
  static std::atomic<uint64_t> attr_done{0};
  const auto kernel = &decode_f32_kernel<DP, NQ, PIECES>;
  hipError_t e = set_max_dynamic_lds_once(attr_done, reinterpret_cast<const void*>(kernel), f32_smem_bytes<DP>());
  if (e != hipSuccess) return e;
  const int heads = PIECES ? a.n_g : a.Hkv, cols = PIECES ? a.n_cols : a.cols;
  dim3 grid((unsigned)(a.n_chunks * heads), (unsigned)((cols + 16 * NQ - 1) / (16 * NQ)), (unsigned)n_z);
  return launch_with(kernel, grid, dim3(256), f32_smem_bytes<DP>(), s, a);
}

// Query columns per workgroup, 16 NQ: a tile costs a workgroup NQ times the matrix work, and the more columns
// it takes the fewer workgroups share that work out.  Microseconds: 4 for a workgroup's start and end, 0.85 for
// 64 rows x 16 columns at head dimension 128; as many workgroups on a CU as tiles fit LDS.  Sync block with 64
// (32 beyond 128 elements) columns throughout and with this rule: 5 x 200..1500 rows, 8/2 heads of 64 13.8 -> 10.9 us,
// 2 x 1500 rows, 24/1 heads of 128 19.0 -> 11.6 (NQ = 1); 8 x 1000..4000 rows, 8/2 heads of 128 31.2 -> 23.3 (NQ = 2,
// 26.4 with 1); 32 x 500..1500 rows, 8/1 heads of 128 112 (NQ = 4, 116 with 2, 140 with 1).
template <int DP>
hipError_t launch_decode_f32_d(const DecodeArgs& a, bool pieces, int n_z, hipStream_t s) {
  constexpr int kMost = DP > 128 ? 2 : 4;
  if (pieces) return launch_decode_f32_t<DP, kMost, true>(a, n_z, s);   // hundreds of columns
  constexpr int kResident = 160 * 1024 / f32_smem_bytes<DP>() > 2 ? 2 : 160 * 1024 / f32_smem_bytes<DP>();
  const double tiles = (a.chunk_rows + kKvTile - 1) / kKvTile, u = 0.85 * DP / 128;
  int nq = 1;
  double best = 1e30;
  for (int x = a.cols <= 16 ? 1 : kMost; x >= 1; x /= 2) {
    const double wgs = (double)a.n_chunks * a.Hkv * ((a.cols + 16 * x - 1) / (16 * x)) * n_z;
    const double places = wgs / ((double)a.n_cus * kResident);
    const double us = 4 * (places > 1 ? places : 1) + ceil(wgs / a.n_cus) * tiles * x * u;
    if (us < best) {
      best = us;
      nq = x;
    }
  }
  if (nq == 1) return launch_decode_f32_t<DP, 1>(a, n_z, s);
  if (nq == 2) return launch_decode_f32_t<DP, 2>(a, n_z, s);
  return launch_decode_f32_t<DP, kMost>(a, n_z, s);
}

}  // namespace

hipError_t launch_decode_f32(const DecodeArgs& a, bool pieces, int n_z, hipStream_t s) {
  if (a.D <= 32) return launch_decode_f32_d<32>(a, pieces, n_z, s);
  if (a.D <= 64) return launch_decode_f32_d<64>(a, pieces, n_z, s);
  if (a.D <= 96) return launch_decode_f32_d<96>(a, pieces, n_z, s);
  if (a.D <= 128) return launch_decode_f32_d<128>(a, pieces, n_z, s);
  if (a.D <= 192) return launch_decode_f32_d<192>(a, pieces, n_z, s);
  return launch_decode_f32_d<256>(a, pieces, n_z, s);
}

}  // namespace fedattn
