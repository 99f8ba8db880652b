// Session reconstruction from block hashes (App. A).
//
// Paper: a request is the follow-up of an earlier request of the same user when its turn is
// larger by one and its block-hash sequence starts with the other's; chained together, such
// requests form a session.  Readings (smetric.h): requests in arrival order; the most recent
// qualifying request is the parent; the empty sequence is a prefix of every sequence; the
// session is the index of the chain's first request.
//
// Mapping to gfx950: a data-parallel join on one small hash table (two slots per request,
// L2-resident at trace sizes):
//   offer   one thread per request p: the slot of (user, turn + 1, block count, last key)
//           holds p (every request gets its own slot: no merging, one CAS per claim);
//   query   one wavefront per request r, lanes over its prefix lengths n = 0 .. nb_r: the
//           slots of (user_r, turn_r, n, key_r[n-1]) give the earlier requests whose whole
//           sequence is r's first n keys -- with chained keys (key j determines blocks 0..j)
//           one key comparison is the whole prefix test; the largest p < r wins;
//           Most lengths have no offer: up to FILT_MAX_REQ requests of FILT_MEAN blocks or
//           more a bitmap of the offers in LDS turns them away (one random 16-byte read per
//           key made the join bound by the L2's lines);
//   roots   one launch: every request follows the jumps, shortening its own for the others
//           as it goes, to its chain's first request.
#include "common.h"

namespace smk {
namespace {

constexpr int TB = 256;

struct OfferSlot {
  uint64_t h;  // 0 = free; the triple's hash | 1 otherwise
  int32_t p;
  int32_t pad;
};

__device__ __forceinline__ uint64_t triple_hash(uint32_t user, int64_t turn, int64_t n, uint64_t last) {
  uint64_t x = mix64(last ^ 0x9E3779B97F4A7C15ull);
  x = mix64(x ^ (uint64_t(user) << 32 | uint32_t(turn)));
  x = mix64(x ^ uint64_t(n) * 0xC2B2AE3D27D4EB4Full);
  return x | 1;
}

__device__ __forceinline__ bool range_ok(const int64_t *blk_off, int32_t r, int64_t n_blocks, int64_t &b0,
                                         int64_t &nb) {
  b0 = blk_off[r];
  const int64_t b1 = blk_off[r + 1];
  nb = b1 - b0;
  return b0 >= 0 && b0 <= b1 && b1 <= n_blocks;
}

// The offers' bitmap: `words` 32-bit words, a power of two, in the session array until the
// roots are written there; an offer sets two bits of one word.  Keys are hashes already, so
// a few 32-bit operations spread them.  One length in six passes at FILT_MAX_REQ requests,
// one in sixty at 32,768.
constexpr int32_t FILT_MAX_REQ = 1 << 17;
// Shorter prompts give a wavefront one lookup per lane, and with the bitmap fewer of them
// wait for theirs at once.  The query without / with it: 131,072 requests of 16 blocks 101 /
// 123 us, of 63 145 / 166, of 100 239 / 221; 34,000 of 16 18 / 25, of 63 25 / 30, of 100 35 / 36, of
// 200 59 / 41; 100,000 of none in one chain 50 / 90.
constexpr int64_t FILT_MEAN = 64;
constexpr uint32_t FILT_MAX_WORDS = 1u << 14;  // 64 KB of LDS, two workgroups to a compute unit
__device__ __forceinline__ uint32_t filt_base(uint32_t user, uint32_t turn) {
  return user * 0x9E3779B1u + turn * 0x85EBCA6Bu;
}
struct FiltBits {
  uint32_t word, bits;
};
__device__ __forceinline__ FiltBits filt_bits(uint32_t base, uint32_t n, uint64_t last, uint32_t words) {
  const uint32_t x = (uint32_t(last) ^ base) + n * 0xC2B2AE35u, y = x ^ (x >> 15) ^ uint32_t(last >> 32);
  return {(y >> 10) & (words - 1), (1u << (y & 31)) | (1u << ((y >> 5) & 31))};
}

__global__ void offer_clear_kernel(OfferSlot *t, uint64_t ns, uint32_t *filt, uint32_t words) {
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  const uint64_t t0 = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  for (uint64_t i = t0; i < ns; i += stride) t[i] = OfferSlot{0, 0, 0};
  for (uint64_t i = t0; i < words; i += stride) filt[i] = 0;
}

__global__ __launch_bounds__(TB) void offer_kernel(const uint64_t *__restrict__ keys, const int64_t *__restrict__ blk_off,
                                                   int32_t n_req, int64_t n_blocks, const uint32_t *__restrict__ user,
                                                   const int32_t *__restrict__ turn, OfferSlot *t, uint64_t ns,
                                                   uint32_t *filt, uint32_t words, int32_t *status) {
  const int32_t p = int32_t(blockIdx.x) * TB + threadIdx.x;
  if (p >= n_req) return;
  int64_t b0, nb;
  if (!range_ok(blk_off, p, n_blocks, b0, nb) || turn[p] < 0) {
    if (status) atomicCAS(status, 0, SMETRIC_EINVAL);
    return;
  }
  const uint64_t last = nb > 0 ? keys[b0 + nb - 1] : 0;
  const uint64_t h = triple_hash(user[p], int64_t(turn[p]) + 1, nb, last);
  if (words) {
    const FiltBits f = filt_bits(filt_base(user[p], uint32_t(turn[p]) + 1), uint32_t(nb), last, words);
    atomicOr(&filt[f.word], f.bits);
  }
  uint64_t s = h & (ns - 1);
  for (uint64_t step = 0; step < ns; ++step, s = (s + 1) & (ns - 1)) {
    if (atomicCAS(reinterpret_cast<unsigned long long *>(&t[s].h), 0ull, h) == 0ull) {
      t[s].p = p;
      return;
    }
  }
}

// The latest earlier request that offered (user, turn, n, last); at most `r` and above `best`.
__device__ __forceinline__ int32_t find_offer(const uint64_t *keys, const int64_t *blk_off, const uint32_t *user,
                                              const int32_t *turn, const OfferSlot *t, uint64_t ns, int32_t r,
                                              uint32_t u, int32_t tr, int64_t n, uint64_t last, int32_t best) {
  const uint64_t h = triple_hash(u, tr, n, last);
  uint64_t s = h & (ns - 1);
  for (uint64_t step = 0; step < ns; ++step, s = (s + 1) & (ns - 1)) {
    const uint64_t sh = t[s].h;
    if (sh == 0) break;
    if (sh != h) continue;
    const int32_t p = t[s].p;
    if (p >= r || p <= best) continue;
    // verify the triple itself (the hash is only a filter)
    const int64_t pb0 = blk_off[p], pnb = blk_off[p + 1] - pb0;
    if (user[p] == u && int64_t(turn[p]) + 1 == tr && pnb == n && (n == 0 || keys[pb0 + n - 1] == last)) best = p;
  }
  return best;
}

// FILT: workgroups of 1024 that keep the bitmap in LDS and take request after request; a lane
// tests QU lengths, their keys loaded together, and looks up those that pass together at the
// end of the stretch.  34,000 requests of some 370 blocks: 74 us (91 us with one bit an offer), 130 us
// as below.  Else a wavefront per request, every length looked up.
constexpr int QT = 1024, QU = 8;
template <bool FILT>
__global__ __launch_bounds__(FILT ? QT : TB) void query_kernel(
    const uint64_t *__restrict__ keys, const int64_t *__restrict__ blk_off, int32_t n_req, int64_t n_blocks,
    const uint32_t *__restrict__ user, const int32_t *__restrict__ turn, const OfferSlot *__restrict__ t, uint64_t ns,
    const uint32_t *__restrict__ filt, uint32_t words, int32_t *__restrict__ parent, int32_t *__restrict__ jump) {
  __shared__ uint32_t bits[FILT ? FILT_MAX_WORDS : 1];
  constexpr int WAVES = (FILT ? QT : TB) / 64;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (FILT) {
    for (uint32_t i = threadIdx.x; i < words; i += QT) bits[i] = filt[i];
    __syncthreads();
  }
  for (int64_t r64 = int64_t(blockIdx.x) * WAVES + wave; r64 < n_req; r64 += int64_t(gridDim.x) * WAVES) {
    const int32_t r = int32_t(r64);
    int64_t b0, nb;
    const int32_t tr = turn[r];
    if (!range_ok(blk_off, r, n_blocks, b0, nb) || tr < 0) {
      if (lane == 0) {
        parent[r] = -1;
        jump[r] = -1;
      }
      continue;
    }
    const uint32_t u = user[r];
    int32_t best = -1;
    if (tr > 0) {
      if (FILT) {
        const uint32_t base = filt_base(u, uint32_t(tr));
        for (int64_t n0 = lane; n0 <= nb + lane; n0 += 64 * QU) {  // whole wavefronts iterate together
          uint64_t last[QU];
#pragma unroll
          for (int j = 0; j < QU; ++j) {
            const int64_t n = n0 + 64 * j;  // prefix length n: blocks 0 .. n-1
            last[j] = n > 0 && n <= nb ? keys[b0 + n - 1] : 0;
          }
          uint32_t cand = 0;
#pragma unroll
          for (int j = 0; j < QU; ++j) {
            const int64_t n = n0 + 64 * j;
            const FiltBits f = filt_bits(base, uint32_t(n), last[j], words);
            cand |= uint32_t(n <= nb && (bits[f.word] & f.bits) == f.bits) << j;
          }
          while (cand) {
            const int j = __ffs(cand) - 1;
            cand &= cand - 1;
            const int64_t n = n0 + 64 * j;
            best = find_offer(keys, blk_off, user, turn, t, ns, r, u, tr, n, n > 0 ? keys[b0 + n - 1] : 0, best);
          }
        }
      } else {
        for (int64_t n = lane; n <= nb; n += 64)
          best = find_offer(keys, blk_off, user, turn, t, ns, r, u, tr, n, n > 0 ? keys[b0 + n - 1] : 0, best);
      }
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) {
        const int32_t o = __shfl_xor(best, m, 64);
        best = o > best ? o : best;
      }
    }
    if (lane == 0) {
      parent[r] = best;
      jump[r] = best >= 0 ? best : r;
    }
  }
}

// Every request follows jump to its chain's first (jump[a] == a; invalid requests are -1),
// writing each jump that it reaches over its own, so that the requests behind it go further
// a step: some ceil(log2 length) steps where the chain runs together.  Any value a jump has
// ever held is an ancestor, lower than its request: an old one costs a step and no more, and
// every walk ends.  (34,000 requests in chains of 8: 5 us;
// a launch per round of doubling, 17 of them: 80 us.)
__global__ __launch_bounds__(TB) void roots_kernel(int32_t *jump, int32_t *__restrict__ session, int32_t n_req) {
  const int32_t r = int32_t(blockIdx.x) * TB + threadIdx.x;
  if (r >= n_req) return;
  int32_t a = __hip_atomic_load(&jump[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  while (a >= 0) {
    const int32_t b = __hip_atomic_load(&jump[a], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (b == a) break;
    __hip_atomic_store(&jump[r], b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    a = b;
  }
  session[r] = a;
}

uint64_t offer_slots(int32_t n_req) {
  uint64_t ns = 64;
  while (ns < 2 * uint64_t(n_req < 1 ? 1 : n_req)) ns <<= 1;
  return ns;
}

// Workspace: the offer table, then one int32 per request for pointer jumping.
uint64_t jump_offset(int32_t n_req) { return (offer_slots(n_req) * sizeof(OfferSlot) + 255) / 256 * 256; }
uint64_t sessions_ws_bytes(int32_t n_req) {
  return jump_offset(n_req) + (uint64_t(n_req < 1 ? 1 : n_req) * 4 + 255) / 256 * 256;
}

}  // namespace
}  // namespace smk

using namespace smk;

extern "C" int smetric_sessions_ws_bytes(int32_t n_req, uint64_t *ws_bytes) {
  if (n_req < 0 || !ws_bytes) return SMETRIC_EINVAL;
  *ws_bytes = sessions_ws_bytes(n_req);
  return SMETRIC_OK;
}

extern "C" int smetric_sessions(const uint64_t *keys, const int64_t *blk_off, int32_t n_req, int64_t n_blocks,
                                const uint32_t *user, const int32_t *turn, int32_t *parent, int32_t *session,
                                int32_t *status, void *workspace, uint64_t ws_bytes, hipStream_t stream) {
  if (n_req < 0 || n_blocks < 0) return SMETRIC_EINVAL;
  if (n_req == 0) return SMETRIC_OK;
  if (!blk_off || !user || !turn || !parent || !session || (n_blocks > 0 && !keys)) return SMETRIC_EINVAL;
  const uint64_t need = sessions_ws_bytes(n_req);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) || ws_bytes < need) return SMETRIC_EWORKSPACE;
  const uint64_t ns = offer_slots(n_req);
  char *base = static_cast<char *>(workspace);
  OfferSlot *t = reinterpret_cast<OfferSlot *>(base);
  int32_t *jump = reinterpret_cast<int32_t *>(base + jump_offset(n_req));
  const int rgrid = (n_req + TB - 1) / TB;
  uint32_t *filt = reinterpret_cast<uint32_t *>(session);
  uint32_t words = 0;  // the bitmap's, 0: none
  // session may be the memory of another array of the call, read until the roots are
  // written: no bitmap there then
  const uint64_t n4 = 4 * uint64_t(n_req);
  const uintptr_t s0 = reinterpret_cast<uintptr_t>(session), s1 = s0 + n4;
  auto apart = [&](const void *p, uint64_t bytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    return !bytes || a >= s1 || a + bytes <= s0;
  };
  if (n_req <= FILT_MAX_REQ && n_blocks / n_req >= FILT_MEAN && apart(keys, 8 * uint64_t(n_blocks)) && apart(blk_off, 2 * n4 + 8) && apart(user, n4) &&
      apart(turn, n4) && apart(parent, n4))
    for (words = 1; 2 * words <= uint32_t(n_req) && words < FILT_MAX_WORDS;) words *= 2;
  hipLaunchKernelGGL(offer_clear_kernel, dim3(int((ns + TB - 1) / TB < 4096 ? (ns + TB - 1) / TB : 4096)), dim3(TB), 0,
                     stream, t, ns, filt, words);
  hipLaunchKernelGGL(offer_kernel, dim3(rgrid), dim3(TB), 0, stream, keys, blk_off, n_req, n_blocks, user, turn, t, ns,
                     filt, words, status);
  const int qw = (n_req + QT / 64 - 1) / (QT / 64);
  if (words)
    hipLaunchKernelGGL(query_kernel<true>, dim3(qw < 512 ? qw : 512), dim3(QT), 0, stream, keys, blk_off, n_req,
                       n_blocks, user, turn, t, ns, filt, words, parent, jump);
  else
    hipLaunchKernelGGL(query_kernel<false>, dim3((n_req + TB / 64 - 1) / (TB / 64)), dim3(TB), 0, stream, keys,
                       blk_off, n_req, n_blocks, user, turn, t, ns, filt, words, parent, jump);
  hipLaunchKernelGGL(roots_kernel, dim3(rgrid), dim3(TB), 0, stream, jump, session, n_req);
  return hip_rc(hipGetLastError());
}
