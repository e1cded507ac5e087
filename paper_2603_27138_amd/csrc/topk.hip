// Top-k block selection with residency split (Alg. 1: TopK, then predicted
// blocks minus resident blocks) and the recall plan (Sec. 3.4), one workgroup
// per (sequence, KV head) pair.
#include "select.h"

namespace scout {

constexpr int kMaxK = 1024;  // what check_problem lets through

// AHEAD: the host's work list and the queries it goes with (HostJob) leave in the same launch, by stores to host memory:
// as copies of their own they cost the stream 5 and 10 us behind the selection, for 4 sequences of 8k tokens.
template <int WAVES, int KPL, bool AHEAD>
__global__ __launch_bounds__(WAVES* kWave) void topk_kernel(
    Dims D, const float* __restrict__ scores, const int32_t* __restrict__ table,
    int32_t* __restrict__ sel_all, int32_t* __restrict__ sel_gpu, int32_t* __restrict__ slot_gpu,
    int32_t* __restrict__ n_gpu, int32_t* __restrict__ sel_host, int32_t* __restrict__ n_host, HostJob J) {
  __shared__ __attribute__((aligned(16))) int lds[selector_lds_ints<WAVES>()];
  __shared__ int l_host[AHEAD ? kMaxK : 1];
  const int b = blockIdx.z, pair = grid_pair();  // grid (1, Hkv, B)
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int nb = num_blocks_of(D, b);
  const int k_eff = D.k < nb ? D.k : nb;

  uint32_t key[KPL];
  int slot[KPL];
  float sc[KPL];
  load_scores<WAVES, KPL>(D, scores, table, pair, wave, lane, sc, slot);
  Selector<WAVES, KPL> S{lds, 0, wave};
  S.prepare();
  mask_keys<WAVES, KPL>(nb, wave, lane, sc, key, slot);
  if constexpr (AHEAD) {  // the pair's query rows: contiguous, a multiple of 16 bytes
    const size_t row = (size_t)D.G * J.q_row, at = pair * row;
    for (int t = threadIdx.x * 16; t < (int)row; t += WAVES * kWave * 16)
      *reinterpret_cast<uint4*>(static_cast<char*>(J.q_out) + at + t) =
          *reinterpret_cast<const uint4*>(static_cast<const char*>(J.q) + at + t);
  }

  Mask<KPL> sel{}, gpu;
  if (k_eff > 0) sel = S.best(key, k_eff, false);
#pragma unroll
  for (int r = 0; r < KPL; ++r) gpu.m[r] = sel.m[r] & __ballot(slot[r] >= 0);
  const size_t out0 = (size_t)pair * D.k;
  const int ng = S.emit(sel, gpu, [&](int r, int i, int at, int at_gpu, bool resident) __attribute__((always_inline)) {
    sel_all[out0 + at] = i;
    if (resident) {
      sel_gpu[out0 + at_gpu] = i;
      slot_gpu[out0 + at_gpu] = slot[r];
    } else {
      sel_host[out0 + at - at_gpu] = i;
      if constexpr (AHEAD) l_host[at - at_gpu] = i;
    }
  });
  const int nh = k_eff - ng;
  if constexpr (AHEAD) __syncthreads();
  for (int t = threadIdx.x; t < D.k; t += WAVES * kWave) {
    if (t >= k_eff) sel_all[out0 + t] = -1;
    if (t >= ng) {
      sel_gpu[out0 + t] = -1;
      slot_gpu[out0 + t] = -1;
    }
    if (t >= nh) sel_host[out0 + t] = -1;
    if constexpr (AHEAD) J.sel[out0 + t] = t < nh ? l_host[t] : -1;
  }
  if (threadIdx.x == 0) {
    n_gpu[pair] = ng;
    n_host[pair] = nh;
    if constexpr (AHEAD) J.n[pair] = nh;
  }
}

template <int WAVES, int KPL>
__global__ __launch_bounds__(WAVES* kWave) void recall_kernel(
    Dims D, const float* __restrict__ scores, int32_t* __restrict__ table,
    int32_t* __restrict__ recall_blk, int32_t* __restrict__ recall_slot,
    int32_t* __restrict__ evict_blk, int32_t* __restrict__ n_recall) {
  __shared__ __attribute__((aligned(16))) int lds[selector_lds_ints<WAVES>()];
  __shared__ int freed[kMaxK];  // slots of the evicted blocks, in ascending block order
  const int b = blockIdx.z, pair = grid_pair();  // grid (1, Hkv, B)
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int nb = num_blocks_of(D, b);
  const int k_eff = D.k < nb ? D.k : nb;

  uint32_t key[KPL];
  int slot[KPL];
  float sc[KPL];
  load_scores<WAVES, KPL>(D, scores, table, pair, wave, lane, sc, slot);
  Selector<WAVES, KPL> S{lds, 0, wave};
  S.prepare();
  mask_keys<WAVES, KPL>(nb, wave, lane, sc, key, slot);

  Mask<KPL> top{}, missing, spare;
  if (k_eff > 0) top = S.best(key, k_eff, false);
#pragma unroll
  for (int r = 0; r < KPL; ++r) {
    const uint64_t res = __ballot(slot[r] >= 0);
    missing.m[r] = top.m[r] & ~res;  // important now, but in host memory
    spare.m[r] = res & ~top.m[r];    // resident, not in the current top-k
  }
  int off_m, off_s, n_missing, n_spare;
  S.offsets(missing, spare, off_m, off_s, n_missing, n_spare);
  const int n = n_missing < n_spare ? n_missing : n_spare;

  Mask<KPL> rec{}, evi{};
  if (n > 0) {
    uint32_t kk[KPL];
    if (n == n_missing) {
      rec = missing;
    } else {  // the cache has room for only n of them: best-ranked first
#pragma unroll
      for (int r = 0; r < KPL; ++r) kk[r] = in_mask(missing.m[r]) ? key[r] : 0u;
      rec = S.best(kk, n, false);
    }
    // worst-ranked spare blocks go: lowest score first, equal scores by higher index
#pragma unroll
    for (int r = 0; r < KPL; ++r) kk[r] = in_mask(spare.m[r]) ? ~key[r] : 0u;
    evi = S.best(kk, n, true);
  }
  const size_t out0 = (size_t)pair * D.k;
  int off_r, off_e, n_rec, n_evi;
  S.offsets(rec, evi, off_r, off_e, n_rec, n_evi);
#pragma unroll
  for (int r = 0; r < KPL; ++r) {
    if (in_mask(evi.m[r])) {
      const int i = (wave * KPL + r) * kWave + lane, at = off_e + mbcnt64(evi.m[r]);
      freed[at] = slot[r];
      recall_slot[out0 + at] = slot[r];
      evict_blk[out0 + at] = i;
      table[(size_t)pair * D.max_blocks + i] = -1;
    }
    off_e += __popcll(evi.m[r]);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < KPL; ++r) {
    if (in_mask(rec.m[r])) {
      const int i = (wave * KPL + r) * kWave + lane, at = off_r + mbcnt64(rec.m[r]);
      recall_blk[out0 + at] = i;
      table[(size_t)pair * D.max_blocks + i] = freed[at];
    }
    off_r += __popcll(rec.m[r]);
  }
  for (int t = threadIdx.x; t < D.k; t += WAVES * kWave) {
    if (t >= n) {
      recall_blk[out0 + t] = -1;
      recall_slot[out0 + t] = -1;
      evict_blk[out0 + t] = -1;
    }
  }
  if (threadIdx.x == 0) n_recall[pair] = n;
}

// ------------------------------------------------------------ host launchers

// Waves per pair and keys per lane by row length.  Few keys per lane and many waves win although the
// waves then exchange through LDS: a wave with 16 keys per lane issues its ballots one after the
// other (1024 blocks: 4.6 us with 8 waves x 2 keys against 8.9 us with one wave x 16; 4096 blocks:
// 6.0 us with 16 waves x 4 against 9.3 us with 4 waves x 16).

#define SCOUT_TOPK(WAVES, KPL) topk_kernel<WAVES, KPL, false>
#define SCOUT_TOPK_AHEAD(WAVES, KPL) topk_kernel<WAVES, KPL, true>
#define SCOUT_RECALL(WAVES, KPL) recall_kernel<WAVES, KPL>
#define SCOUT_TOPK_DISPATCH(KERNEL, ...)                                                     \
  do {                                                                                       \
    if (D.B == 0) return SCOUT_OK;                                                           \
    dim3 grid(1, D.Hkv, D.B);                                                                \
    if (D.max_blocks <= 256)                                                                 \
      hipLaunchKernelGGL((KERNEL(1, 4)), grid, dim3(kWave), 0, st, __VA_ARGS__);             \
    else if (D.max_blocks <= 1024)                                                           \
      hipLaunchKernelGGL((KERNEL(8, 2)), grid, dim3(8 * kWave), 0, st, __VA_ARGS__);         \
    else if (D.max_blocks <= 4096)                                                           \
      hipLaunchKernelGGL((KERNEL(16, 4)), grid, dim3(16 * kWave), 0, st, __VA_ARGS__);       \
    else if (D.max_blocks <= 16384)                                                          \
      hipLaunchKernelGGL((KERNEL(16, 16)), grid, dim3(16 * kWave), 0, st, __VA_ARGS__);      \
    else                                                                                     \
      return SCOUT_EUNSUPPORTED;                                                             \
  } while (0)

int launch_topk(const Dims& D, const float* scores, const int32_t* table, int32_t* sel_all,
                int32_t* sel_gpu, int32_t* slot_gpu, int32_t* n_gpu, int32_t* sel_host,
                int32_t* n_host, const HostJob* job, hipStream_t st) {
  if (job != nullptr)
    SCOUT_TOPK_DISPATCH(SCOUT_TOPK_AHEAD, D, scores, table, sel_all, sel_gpu, slot_gpu, n_gpu, sel_host, n_host, *job);
  else
    SCOUT_TOPK_DISPATCH(SCOUT_TOPK, D, scores, table, sel_all, sel_gpu, slot_gpu, n_gpu, sel_host, n_host, HostJob{});
  return hipGetLastError() == hipSuccess ? SCOUT_OK : SCOUT_EHIP;
}

int launch_recall(const Dims& D, const float* scores, int32_t* table, int32_t* recall_blk,
                  int32_t* recall_slot, int32_t* evict_blk, int32_t* n_recall, hipStream_t st) {
  SCOUT_TOPK_DISPATCH(SCOUT_RECALL, D, scores, table, recall_blk, recall_slot, evict_blk, n_recall);
  return hipGetLastError() == hipSuccess ? SCOUT_OK : SCOUT_EHIP;
}

}  // namespace scout
