// Decode append: the key and value of the token that decode just produced join the cache, and the
// digest of the block they fall into (Sec. 2.2: channel-wise min/max over the block's keys, or their
// sum for mean pooling) is kept up to date, so that the digests of all blocks stay on the GPU as Sec. 3.2 requires while the
// sequence grows.
//
// One workgroup per sequence, one thread per four channels of a KV head: a few kilobytes per call, bound by latency,
// not by bandwidth: the length, then the table entry and the digest at that length, then the stores.  The new rows
// are requested together with the length.  The length is advanced in place as soon as every wave has read it: a
// barrier in front of that store with the rows' stores ahead of it would wait until those are acknowledged, one more trip.
#include "common.h"

namespace scout {

constexpr int kAppendVec = 4;  // channels per thread

// Four consecutive elements of storage type as they lie in memory.
template <int DT>
struct Vec4 {
  typedef uint32_t word __attribute__((ext_vector_type(DT == SCOUT_BF16 ? 2 : 4)));
  word w;
  static __device__ __forceinline__ Vec4 load(const void* base, size_t elem) {
    return Vec4{*reinterpret_cast<const word*>(static_cast<const char*>(base) + elem * (DT == SCOUT_BF16 ? 2 : 4))};
  }
  __device__ __forceinline__ void store(void* base, size_t elem) const {
    *reinterpret_cast<word*>(static_cast<char*>(base) + elem * (DT == SCOUT_BF16 ? 2 : 4)) = w;
  }
  __device__ __forceinline__ float get(int i) const {
    if constexpr (DT == SCOUT_BF16) return (i & 1) ? bf16_hi(w[i >> 1]) : bf16_lo(w[i >> 1]);
    else return __uint_as_float(w[i]);
  }
  // element i becomes x's element i, bit for bit
  __device__ __forceinline__ void take(int i, const Vec4& x) {
    if constexpr (DT == SCOUT_BF16) {
      const uint32_t m = (i & 1) ? 0xffff0000u : 0x0000ffffu;
      w[i >> 1] = (w[i >> 1] & ~m) | (x.w[i >> 1] & m);
    } else {
      w[i] = x.w[i];
    }
  }
};

template <int DT>
__global__ __launch_bounds__(1024) void append_kernel(Dims D, int32_t* ctx_len, const void* __restrict__ k_new,
                                                     const void* __restrict__ v_new,
                                                     const int32_t* __restrict__ new_slot, void* digest,
                                                     int32_t* block_table, void* k_pool, void* v_pool,
                                                     long long n_slots, void* host_k, void* host_v) {
  using V = Vec4<DT>;
  // every argument in the first trip for arguments: left to itself the compiler fetches those that are used behind the
  // length once the length is there
  asm volatile("" ::"s"(digest), "s"(block_table), "s"(k_pool), "s"(v_pool), "s"(n_slots), "s"(new_slot), "s"(host_k), "s"(host_v),
               "s"(ctx_len), "s"(D.max_blocks), "s"(D.tile_stride), "s"(D.digest_kind), "s"(D.s_shift), "s"(D.S));
  const int b = blockIdx.x;
  const int n = D.Hkv * D.d / kAppendVec, c_shift = D.d == 64 ? 4 : 5;  // threads per KV head: d / 4
  int e = threadIdx.x;
  V k{}, v{};
  auto fetch = [&]() __attribute__((always_inline)) {  // what does not depend on the length
    if (e < n) {
      const size_t row = (size_t)b * D.Hkv * D.d + (size_t)e * kAppendVec;
      k = V::load(k_new, row);
      v = V::load(v_new, row);
    }
  };
  fetch();
  const int t = __builtin_amdgcn_readfirstlane(ctx_len[b]);
  if (t < 0 || t >= D.max_blocks * D.S) return;  // a full sequence is left as it is (the whole workgroup leaves)
  // Every wave has its copy of the length: one thread may advance it now.
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  if (threadIdx.x == 0) ctx_len[b] = t + 1;
  const int j = t >> D.s_shift, r = t & (D.S - 1);  // S and d are powers of two
  while (e < n) {
    const int g = e >> c_shift, c = (e & ((1 << c_shift) - 1)) * kAppendVec;
    const size_t pair = (size_t)b * D.Hkv + g;
    int32_t* entry = block_table + pair * D.max_blocks + j;
    // a block's first token opens it with the slot the caller chose; later tokens follow the table
    const int slot = r == 0 ? new_slot[pair] : *entry;
    if (D.digest_kind == 1) {  // mean pooling: the block's running sum in binary32, one addition per token
      float4* sums = reinterpret_cast<float4*>(static_cast<float*>(digest) + (pair * D.max_blocks + j) * D.d + c);
      float4 x = make_float4(k.get(0), k.get(1), k.get(2), k.get(3));
      if (r != 0) {
        const float4 s = *sums;
        x = make_float4(s.x + x.x, s.y + x.y, s.z + x.z, s.w + x.w);
      }
      *sums = x;
    } else {
      const size_t i_min = ((pair * D.max_blocks + j) * 2) * D.d + c, i_max = i_min + D.d;
      V lo = k, hi = k;
      if (r != 0) {
        lo = V::load(digest, i_min);
        hi = V::load(digest, i_max);
        // strict comparisons: of equal elements the older one stays, as in a first-occurrence min/max
#pragma unroll
        for (int i = 0; i < kAppendVec; ++i) {
          if (k.get(i) < lo.get(i)) lo.take(i, k);
          if (k.get(i) > hi.get(i)) hi.take(i, k);
        }
      }
      lo.store(digest, i_min);
      hi.store(digest, i_max);
    }
    if (slot >= 0 && slot < n_slots) {
      const size_t row = (size_t)slot * D.tile_stride + (size_t)r * D.d + c;
      k.store(k_pool, row);
      v.store(v_pool, row);
    }
    if (host_k != nullptr) {  // the host's copy of every block (pinned memory), whatever the residency: this is what a
                              // later recall reads, and why an eviction has nothing to move
      const size_t row = ((pair * D.max_blocks + j) * D.S + r) * D.d + c;
      k.store(host_k, row);
      v.store(host_v, row);
    }
    if (r == 0 && c == 0) *entry = slot;  // nobody reads the entry in this call when r == 0
    e += blockDim.x;
    fetch();
  }
}

int launch_append(const Dims& D, int dtype, int32_t* ctx_len, const void* k_new, const void* v_new,
                  const int32_t* new_slot, void* digest, int32_t* block_table, void* k_pool, void* v_pool,
                  long long n_slots, void* host_k, void* host_v, hipStream_t st) {
  if (D.B == 0) return SCOUT_OK;
  // all of a sequence's row at once where it fits a workgroup: the call should walk its chain of trips once
  const int threads = D.Hkv * D.d / kAppendVec;
  const dim3 block(threads >= 1024 ? 1024 : (threads + 63) / 64 * 64);
  if (dtype == SCOUT_BF16)
    hipLaunchKernelGGL(append_kernel<SCOUT_BF16>, dim3(D.B), block, 0, st, D, ctx_len, k_new, v_new, new_slot,
                       digest, block_table, k_pool, v_pool, n_slots, host_k, host_v);
  else
    hipLaunchKernelGGL(append_kernel<SCOUT_F32>, dim3(D.B), block, 0, st, D, ctx_len, k_new, v_new, new_slot,
                       digest, block_table, k_pool, v_pool, n_slots, host_k, host_v);
  return hipGetLastError() == hipSuccess ? SCOUT_OK : SCOUT_EHIP;
}

}  // namespace scout
