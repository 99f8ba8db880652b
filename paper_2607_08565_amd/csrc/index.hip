// Global block index in HBM: layout, insert (K2 + K7), evict (K6), dump, stats.
//
// Paper: the router consults each instance's local KV$ contents ("kvc", Sec. 4.1) to get
// the prefix hit c_i; the structure is not described.  The index here is the set of
// entries (key, instance) with the producing session and the last epoch; after a batch
// is routed every full block of each prompt is entered on its target (the target's
// prefill caches the prompt, Sec. 2 and 4.2), and a fraction of the oldest entries can be
// evicted (local tiers evict, Sec. 2 and 4.2 "session_cached").
//
// Layout of the caller's buffer:
//   [0, 256)                 IndexHdr: entry count, sticky status, pool use
//   slots                    n_buckets x 128 B: keys[8] then values[8]
//   pool                     n_records x bitmap_words x 8 B: holder bitmaps
//   masks                    n_buckets x 16 bits: each chain start's displacement mask
// A key normally owns one PLAIN slot per holder in its home chain (linear probing over
// buckets from home_bucket(key)).  When a key gains more than T holders its plain slots
// are replaced by one HEADER slot pointing at a bitmap record, and every holder becomes a
// MEMBER slot found from member_bucket(key, inst); probes of the key then read one
// bucket line plus the bitmap instead of walking T+ slots.  If the pool runs out, keys
// simply stay plain.  Slots are only ever claimed (EMPTY -> key by compare-and-swap) or
// turned into tombstones, so every slot of a key lies before the first EMPTY slot of its
// chain.  Eviction selects the oldest entries by (epoch, key, instance) digit by digit
// among those that one scan finds near the cut, then turns them into tombstones in place, or --
// once tombstones would take too many slots -- rebuilds the table from the survivors.
//
// Insert pipeline (no sort, no host synchronisation):
//   clear      scratch dedupe table
//   find       per pair (r, j): validate; find (key, target) -> refresh position, or
//              enter the pair in the dedupe table keyed by (key, instance), keeping the
//              lowest request index (atomic min); the first to enter a pair places it.  The
//              last workgroup checks: first error -> EINVAL/EFULL, nothing changes; else count
//   apply      epoch = max(old, epoch) for existing entries; each distinct new pair claims a
//              slot, and the thread whose slot becomes the key's (T+1)-th plain slot --
//              unique, since claims fill a chain in order -- queues the key for conversion
//   spill      queued keys get a bitmap record, member slots, a header and tombstones
// Batches of at most SI_LINE or SI_MAX blocks take one launch (ins_small_kernel); a probed batch past
// the direct form's size takes the region-ordered passes.
#include <rocprim/device/device_radix_sort.hpp>

#include <time.h>
#include <unistd.h>

#include "common.h"

namespace smk {

uint64_t process_owner() {
  static const uint64_t owner = [] {
    static char here;
    timespec t{};
    clock_gettime(CLOCK_REALTIME, &t);
    uint64_t x = mix64(uint64_t(t.tv_sec) * 1000000000ull + uint64_t(t.tv_nsec));
    x = mix64(x ^ (uint64_t(getpid()) << 40)) ^ reinterpret_cast<uintptr_t>(&here);
    return mix64(x) | 1;  // 0: an index written before the word was
  }();
  return owner;
}

namespace {

constexpr int TB = 256;
constexpr int MAX_GRID = 4096;

inline uint64_t round_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }
inline int grid_for(uint64_t n) {
  const uint64_t g = (n + TB - 1) / TB;
  return int(g < 1 ? 1 : (g > MAX_GRID ? MAX_GRID : g));
}

__global__ void fill_kernel(uint64_t *p, uint64_t n_words, uint64_t value) {
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n_words; i += stride) p[i] = value;
}

__global__ void set_int_kernel(int *p, int v) { *p = v; }

// An index's slots EMPTY with unset values, its header saying that no entry has an epoch.
__global__ void unset_values_kernel(IndexHdr *h, uint64_t owner, uint64_t *slots, uint64_t n_buckets) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    h->epoch_top = 1;
    h->epoch_owner = owner;
  }
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t b = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; b < n_buckets; b += stride) {
    ulonglong2 *v = reinterpret_cast<ulonglong2 *>(slots + b * BUCKET_WORDS + SLOTS);
#pragma unroll
    for (int i = 0; i < SLOTS / 2; ++i) v[i] = make_ulonglong2(VAL_UNSET, VAL_UNSET);
  }
}

int fill(void *p, uint64_t bytes, uint64_t value, hipStream_t s) {
  const uint64_t n = bytes / 8;
  if (n == 0) return SMETRIC_OK;
  hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n)), dim3(TB), 0, s, static_cast<uint64_t *>(p), n, value);
  return hip_rc(hipGetLastError());
}

struct Layout {
  int32_t words, threshold;
  uint64_t n_records, n_buckets, slots_off, pool_off, bytes;
};

// n_slots = 0: the table holds capacity entries (plus converted keys' headers and
// tombstones) at <= 3/4 occupancy.  Otherwise the caller fixes the slot count (rounded up
// to whole buckets), which must leave at least 1/16 of the slots free at capacity.
bool layout_for(uint64_t capacity, int32_t n_inst, uint64_t n_slots, Layout &L) {
  if (capacity == 0 || capacity > (uint64_t(1) << 40) || n_inst < 1 || n_inst > 65536) return false;
  if (n_slots > (uint64_t(1) << 41)) return false;
  L.words = bitmap_words_for(n_inst);
  L.threshold = threshold_for(n_inst);
  uint64_t rec = capacity / 256;
  if (rec < 64) rec = 64;
  const uint64_t rec_max = capacity / uint64_t(L.threshold + 1) + 1;
  if (rec > rec_max) rec = rec_max;
  L.n_records = rec;
  // slots: live entries plus headers/tombstones of converted keys, at <= 3/4 occupancy
  const uint64_t slots = capacity + uint64_t(L.threshold) * rec;
  if (n_slots == 0) {
    L.n_buckets = (slots * 4 / 3 + SLOTS - 1) / SLOTS + 1;
  } else {
    L.n_buckets = (n_slots + SLOTS - 1) / SLOTS;
    if (slots * 16 > L.n_buckets * SLOTS * 15) return false;
  }
  L.slots_off = sizeof(IndexHdr);
  L.pool_off = L.slots_off + L.n_buckets * BUCKET_WORDS * 8;
  // then the displacement masks, MASK_W bits per bucket (dev_view finds them after the pool)
  L.bytes = round_up(L.pool_off + L.n_records * uint64_t(L.words) * 8 + mask_bytes(L.n_buckets), 256);
  return true;
}

int attach(smetric_index *idx, void *mem, uint64_t mem_bytes, uint64_t capacity, int32_t n_inst, uint64_t n_slots) {
  Layout L;
  if (!idx || !mem || !layout_for(capacity, n_inst, n_slots, L) || mem_bytes < L.bytes ||
      (reinterpret_cast<uintptr_t>(mem) & 255))
    return SMETRIC_EINVAL;
  char *base = static_cast<char *>(mem);
  idx->mem = mem;
  idx->mem_bytes = mem_bytes;
  idx->capacity = capacity;
  idx->n_instances = n_inst;
  idx->bitmap_words = L.words;
  idx->spill_threshold = L.threshold;
  idx->reserved0 = 0;
  idx->n_buckets = L.n_buckets;
  idx->n_records = L.n_records;
  idx->slots = reinterpret_cast<uint64_t *>(base + L.slots_off);
  idx->pool = reinterpret_cast<uint64_t *>(base + L.pool_off);
  idx->hdr = base;
  return SMETRIC_OK;
}

// ---------------------------------------------------------------------------------
// Table primitives
// ---------------------------------------------------------------------------------
struct Found {
  int64_t slot;  // bucket * SLOTS + s, or -1
  uint64_t val;
};

// Find the entry (key, inst), looking through a bitmap record when the key has one.
__device__ Found find_member(const DevIndex &ix, uint64_t key, uint32_t inst) {
  ChainWalk w = chain_start(member_bucket(key, inst, ix.n_buckets, ix.nb_inv), member_cls(key, inst));
  bool had_empty;
  do {
    const uint64_t m = w.b;
    const uint64_t *mk = ix.slots + m * BUCKET_WORDS;
    const BucketScan sc = scan_bucket(mk, key);
    uint32_t mm = sc.match;
    while (mm) {
      const int t = __builtin_ctz(mm);
      mm &= mm - 1;
      const uint64_t v = mk[SLOTS + t];
      if (val_kind(v) == MEMBER && val_inst(v) == inst) return Found{int64_t(m * SLOTS + t), v};
    }
    had_empty = sc.empty != 0;
  } while (chain_next(ix, w, had_empty));
  return Found{-1, 0};
}

// The entry (key, inst) of a key with bitmap record rec.
__device__ __forceinline__ Found find_holder(const DevIndex &ix, uint64_t rec, uint64_t key, uint32_t inst) {
  const uint64_t bw = ix.pool[rec * uint64_t(ix.words) + (inst >> 6)];
  if (!((bw >> (inst & 63)) & 1)) return Found{-1, 0};
  return find_member(ix, key, inst);
}

__device__ Found find_entry(const DevIndex &ix, uint64_t key, uint32_t inst) {
  ChainWalk w = chain_start(home_bucket(key, ix.n_buckets), key_cls(key));
  bool had_empty;
  do {
    const uint64_t b = w.b;
    const uint64_t *bk = ix.slots + b * BUCKET_WORDS;
    const BucketScan sc = scan_bucket(bk, key);
    uint32_t mm = sc.match;
    while (mm) {
      const int s = __builtin_ctz(mm);
      mm &= mm - 1;
      const uint64_t v = bk[SLOTS + s];
      const uint32_t kind = val_kind(v);
      if (kind == PLAIN && val_inst(v) == inst) return Found{int64_t(b * SLOTS + s), v};
      if (kind == HEADER) return find_holder(ix, val_rec(v), key, inst);
    }
    had_empty = sc.empty != 0;
  } while (chain_next(ix, w, had_empty));
  return Found{-1, 0};
}

__device__ __forceinline__ uint64_t *val_ptr(const DevIndex &ix, int64_t slot) {
  return ix.slots + (slot / SLOTS) * BUCKET_WORDS + SLOTS + (slot % SLOTS);
}

// Walk the chain from bucket b and claim its first EMPTY slot for `key`.  With
// want_header, stop instead at a HEADER slot of `key` (the key has a bitmap record).
// `same` counts slots holding `key` ahead of the claimed one.  Plain loads may see a
// stale EMPTY; the compare-and-swap then fails and returns the slot's real key, and
// slots never return to EMPTY, so the count is exact.
// With max_same, the walk gives up (capped) once it has seen max_same slots of `key`
// ahead of any free slot: that key is about to get a bitmap record, and its remaining
// new holders are entered after the conversion instead of piling up plain slots that
// would all turn into tombstones.
// With want_inst, a PLAIN slot of (key, want_inst) met on the way ends the walk instead
// (existing): the pair is already an entry.
struct Claim {
  int64_t slot;      // claimed slot, or -1
  int64_t header;    // HEADER slot of key when found, else -1
  int64_t existing;  // PLAIN slot of (key, want_inst) when found, else -1
  uint32_t same;
  bool capped;
};
constexpr uint32_t NO_INST = 0xFFFFFFFFu;
__device__ Claim claim_slot(const DevIndex &ix, uint64_t b, uint64_t key, uint32_t cls, bool want_header,
                            uint32_t max_same = 0xFFFFFFFFu, uint32_t want_inst = NO_INST) {
  Claim c{-1, -1, -1, 0, false};
  const uint64_t h = b;  // the chain start whose displacement mask records the claim
  for (uint64_t step = 0; step < ix.n_buckets; ++step, b = next_bucket(b, ix.n_buckets)) {
    uint64_t *bk = ix.slots + b * BUCKET_WORDS;
    const BucketScan sc = scan_bucket(bk, key);
    if (want_header || want_inst != NO_INST) {
      uint32_t mm = sc.match;
      while (mm) {
        const int s = __builtin_ctz(mm);
        mm &= mm - 1;
        const uint64_t v = bk[SLOTS + s];
        if (want_header && val_kind(v) == HEADER) {
          c.header = int64_t(b * SLOTS + s);
          return c;
        }
        if (val_kind(v) == PLAIN && val_inst(v) == want_inst) {
          c.existing = int64_t(b * SLOTS + s);
          return c;
        }
      }
    }
    if (!sc.empty) {
      c.same += __popc(sc.match);
      if (c.same >= max_same) {
        c.capped = true;
        return c;
      }
      continue;
    }
    // slots before the first EMPTY are final; try the EMPTY ones in order
    const int first = __builtin_ctz(sc.empty);
    c.same += __popc(sc.match & ((1u << first) - 1u));
    for (int s = first; s < SLOTS; ++s) {
      if (c.same >= max_same) {
        c.capped = true;
        return c;
      }
      const uint64_t k = atomicCAS(reinterpret_cast<unsigned long long *>(&bk[s]), KEY_EMPTY, key);
      if (k == KEY_EMPTY) {
        c.slot = int64_t(b * SLOTS + s);
        mask_note(ix, h, b, cls);
        return c;
      }
      if (k == key) {  // claimed meanwhile by another pair of the same key (never this pair)
        if (want_header && val_kind(__hip_atomic_load(&bk[SLOTS + s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == HEADER) {
          c.header = int64_t(b * SLOTS + s);  // cannot happen: headers predate this kernel
          return c;
        }
        ++c.same;
      }
    }
  }
  return c;
}

// epoch = max(old, epoch) of the entry at `slot` (kind and instance given), session kept
// (an existing pair).
__device__ __forceinline__ void refresh_at(const DevIndex &ix, int64_t slot, uint32_t kind, uint32_t inst,
                                           uint32_t epoch) {
  raise_epoch_at(val_ptr(ix, slot), kind, inst, epoch);
}

// Enter a pair that is not known to be an entry (one per pair and call: pairs are
// distinct).  Returns PLACED, REFRESHED (it was an entry: its epoch is raised instead),
// DEFERRED (capped: enter it again after the key's conversion, uncapped) or FAILED (no
// free slot).  trigger is set when the slot is the key's (T+1)-th plain slot, the last
// one a key gets before its conversion.
enum Placed { PLACED = 0, DEFERRED = 1, FAILED = 2, REFRESHED = 3 };
__device__ int place_new(const DevIndex &ix, uint64_t key, uint32_t inst, uint32_t epoch, uint32_t sess,
                         bool &trigger, bool capped) {
  trigger = false;
  const Claim c = claim_slot(ix, home_bucket(key, ix.n_buckets), key, key_cls(key), true,
                             capped ? uint32_t(ix.threshold) + 1 : 0xFFFFFFFFu, inst);
  if (c.existing >= 0) {
    refresh_at(ix, c.existing, PLAIN, inst, epoch);
    return REFRESHED;
  }
  if (c.header >= 0) {
    const uint64_t rec = val_rec(*val_ptr(ix, c.header));
    const unsigned long long old = atomicOr(
        reinterpret_cast<unsigned long long *>(&ix.pool[rec * uint64_t(ix.words) + (inst >> 6)]), 1ull << (inst & 63));
    if ((old >> (inst & 63)) & 1) {  // already a member
      const Found f = find_member(ix, key, inst);
      if (f.slot < 0) return FAILED;
      refresh_at(ix, f.slot, MEMBER, inst, epoch);
      return REFRESHED;
    }
    const Claim m = claim_slot(ix, member_bucket(key, inst, ix.n_buckets, ix.nb_inv), key, member_cls(key, inst), false);
    if (m.slot < 0) return FAILED;
    *val_ptr(ix, m.slot) = make_val(inst, MEMBER, epoch, sess);
    return PLACED;
  }
  if (c.capped) return DEFERRED;
  if (c.slot < 0) return FAILED;
  *val_ptr(ix, c.slot) = make_val(inst, PLAIN, epoch, sess);
  trigger = c.same == uint32_t(ix.threshold);
  return PLACED;
}

// Can no entry be above `epoch`?  And the header's bound raised to it, by one thread of an
// insert that goes through, in a kernel after those that ask.
__device__ __forceinline__ bool epoch_tops(const DevIndex &ix, uint32_t epoch) {
  return ix.hdr->epoch_top != 0 && epoch + 1 >= ix.hdr->epoch_top && ix.hdr->epoch_owner == ix.owner;
}
__device__ __forceinline__ void keep_epoch_top(const DevIndex &ix, uint32_t epoch) {
  if (ix.hdr->epoch_top != 0 && epoch + 1 > ix.hdr->epoch_top) ix.hdr->epoch_top = epoch + 1;
}

// A REFRESHED pair was counted as new by the capacity check: take it back, one atomic
// per wavefront.
__device__ __forceinline__ void uncount_refreshed(const DevIndex &ix, bool refreshed) {
  const uint64_t m = __ballot(refreshed);
  if (m && (threadIdx.x & 63) == uint32_t(__builtin_ctzll(m)))
    atomicAdd(&ix.hdr->n_entries, 0ull - (unsigned long long)__popcll(m));
}

// Replace the plain slots of `key` by a bitmap record (one thread per key).
__device__ bool spill_key(const DevIndex &ix, uint64_t key) {
  const unsigned long long rec = atomicAdd(reinterpret_cast<unsigned long long *>(&ix.hdr->rec_used), 1ull);
  if (rec >= ix.n_records) return true;  // pool exhausted: the key stays plain
  uint64_t *bm = ix.pool + rec * uint64_t(ix.words);
  int64_t first = -1;
  uint64_t b = home_bucket(key, ix.n_buckets);
  for (uint64_t step = 0; step < ix.n_buckets; ++step) {
    uint64_t *bk = ix.slots + b * BUCKET_WORDS;
    bool end = false;
    for (int s = 0; s < SLOTS; ++s) {
      const uint64_t k = bk[s];
      if (k == KEY_EMPTY) {
        end = true;
        break;
      }
      if (k != key) continue;
      const uint64_t v = bk[SLOTS + s];
      if (val_kind(v) != PLAIN) continue;
      const uint32_t inst = val_inst(v);
      bm[inst >> 6] |= 1ull << (inst & 63);
      const Claim m = claim_slot(ix, member_bucket(key, inst, ix.n_buckets, ix.nb_inv), key, member_cls(key, inst), false);
      if (m.slot < 0) return false;
      *val_ptr(ix, m.slot) = make_val(inst, MEMBER, val_epoch(v), val_session(v));
      if (first < 0) {
        first = int64_t(b * SLOTS + s);
        bk[SLOTS + s] = header_val(rec);
      } else {
        bk[s] = KEY_TOMB;
      }
    }
    if (end) break;
    b = (b + 1 == ix.n_buckets) ? 0 : b + 1;
  }
  return true;
}

// ---------------------------------------------------------------------------------
// Insert
// ---------------------------------------------------------------------------------
struct WsHdr {
  unsigned long long n_pairs;  // pairs over all request ranges
  unsigned long long n_trig;   // keys queued for conversion
  int err;                     // first input error seen by the probe
  int abort;                   // set by the check: leave the index unchanged
  unsigned long long n_cand;   // pairs absent before the batch (region-ordered insert)
  unsigned long long n_def;    // new pairs deferred until their key's conversion
  unsigned long long nsub;     // region-ordered insert: bins per region (a power of two)
  unsigned long long n_dd2;    // region-ordered insert: fallback pair-table slots in use
  unsigned long long n_over;   // region-ordered insert: candidates in bins too large for LDS
  int inl;                     // region-ordered insert: refreshes done by the classify pass
  int pad1;
  unsigned long long turns;    // find pass: new pairs, workgroups that have ended, errors (ins_check_last)
  unsigned long long pad[22];
};
static_assert(sizeof(WsHdr) == 256, "ws header size");

// Dedupe table slot: the pair's key and (inst + 1) << 32 | lowest request index, both in
// one 16-byte slot so a pair costs one line; all-zero = free.
struct DSlot {
  uint64_t key;
  uint64_t w2;
};
__device__ __forceinline__ uint32_t dd_inst(uint64_t w2) { return uint32_t(w2 >> 32) - 1; }
__device__ __forceinline__ uint32_t dd_req(uint64_t w2) { return uint32_t(w2); }

// Candidate of the region-ordered insert: an absent pair, as it enters the dedupe.
struct Cand {
  uint64_t key;
  uint64_t w2;  // same encoding as DSlot::w2
};

// Distinct new pair of the region-ordered insert, in bin order (key KEY_EMPTY: a dropped
// duplicate).  w2 as in DSlot, or NP_FALLBACK | h: the pair went through the fallback
// pair table and dd[h].w2 holds its final (lowest) request.
struct NewPair {
  uint64_t key;
  uint64_t w2;
};
constexpr uint64_t NP_FALLBACK = uint64_t(1) << 63;
__device__ __forceinline__ uint64_t np_w2(const NewPair &e, const DSlot *dd) {
  return (e.w2 & NP_FALLBACK) ? dd[e.w2 & ~NP_FALLBACK].w2 : e.w2;
}

// Binning of the region-ordered insert's candidates: bins are NREG x nsub equal ranges of
// home buckets, so every candidate of a key -- and of a (key, instance) pair -- lies in
// one bin, and a bin is deduplicated in LDS by one workgroup.
constexpr int KCH = 32;                     // chunks per region of the bin partition
// The classify pass runs INS_WG workgroups (as many as the device holds at its register
// use), each filling one candidate segment.
constexpr int INS_WG = 1024;
// Workgroups of the placement's grid.
constexpr int PLACE_WG = 4096;
inline uint64_t ins_segment(uint64_t n) {
  const uint64_t span = uint64_t(INS_WG) * WG_THREADS;
  return (n + span - 1) / span * WG_THREADS;
}
constexpr int SEG_PER_CH = INS_WG / KCH;    // classify segments per chunk
constexpr int NSUB_MAX = 1024;              // bins per region, at most
constexpr int NBIN_MAX = NREG * NSUB_MAX;
constexpr int BIN_TARGET = 1536;            // nsub keeps the mean bin at or below this
constexpr int DT = 4096;                    // slots of a bin's LDS pair table
constexpr int BIN_CAP = 3072;               // larger bins stream through the LDS pair table
static_assert(INS_WG % KCH == 0 && SEG_PER_CH <= 64, "chunk = whole classify segments");
static_assert(BIN_CAP + WG_THREADS < DT, "an LDS pair table never fills");

// Workgroups of the find and apply passes: at most 2 FIND_WG.
constexpr int FIND_WG = 256;
// Workgroups of the region-ordered insert's first pass, and of its dedupe pass (as many as
// the device holds at its LDS use; each takes a turn on one word, see ins_check_last).
constexpr int HEAD_WG = 64;
constexpr int DEDUPE_WG = 512;

struct InsWs {
  WsHdr *hdr;
  uint64_t *pos;    // per block: slot + 1 of an entry to refresh, a new pair (POS_NEW), 0 = none
  DSlot *dd;        // dedupe table (region-ordered insert: fallback pair table)
  uint64_t *trig;   // keys queued for conversion
  uint64_t *def;    // list positions of deferred new pairs
  Cand *cand;       // region-ordered insert: absent pairs, one segment per workgroup,
                    // cut into one part per region
  uint32_t *cand_cnt;  // [INS_WG] candidates in each segment
  uint32_t *ctot;   // [NREG][KCH] candidates in each chunk of the bin partition
  uint32_t *soff;   // [INS_WG][NREG] offset of each (segment, region) part in its segment
  uint32_t *rcnt;   // [INS_WG][NREG] candidates in each part
  uint32_t *hist2;  // [NREG][KCH][NSUB_MAX] candidates of each bin in each chunk
  uint32_t *base2;  // [NREG][KCH][NSUB_MAX] first bin-order position of each (chunk, bin)
  uint32_t *bstart; // [NBIN_MAX + 1] first bin-order position of each bin
  uint32_t *bad;    // [HEAD_WG] some request's target or session is invalid
  Cand *bcand;      // candidates in bin order
  NewPair *np;      // bin order: distinct new pairs
  uint64_t n_dedupe;
  uint64_t list_cap;  // entries in trig and def
  uint64_t seg;       // segment length of the region-ordered insert
};

uint64_t dedupe_size(int64_t n_blocks) {
  uint64_t n = 64;
  while (n < 2 * uint64_t(n_blocks)) n <<= 1;
  return n;
}

uint64_t insert_ws_layout(int64_t n_blocks, InsWs *ws, void *base) {
  const uint64_t n = uint64_t(n_blocks < 1 ? 1 : n_blocks);
  const uint64_t nd = dedupe_size(n_blocks);
  const uint64_t seg = ins_segment(n), seg_n = seg * INS_WG;
  const uint64_t nl = seg_n > n ? seg_n : n;
  uint64_t off = 0;
  auto take = [&](uint64_t bytes) {
    const uint64_t o = off;
    off = round_up(off + bytes, 256);
    return o;
  };
  const uint64_t o_hdr = take(sizeof(WsHdr));
  const uint64_t o_pos = take(8 * n);
  const uint64_t o_dd = take(16 * nd);
  const uint64_t o_trig = take(8 * nl);
  const uint64_t o_def = take(8 * nl);
  const uint64_t o_cand = take(sizeof(Cand) * seg_n);
  const uint64_t o_cc = take(4ull * INS_WG);
  const uint64_t o_ct = take(4ull * NREG * KCH);
  const uint64_t o_soff = take(4ull * INS_WG * NREG);
  const uint64_t o_rcnt = take(4ull * INS_WG * NREG);
  const uint64_t o_h2 = take(4ull * NREG * KCH * NSUB_MAX);
  const uint64_t o_b2 = take(4ull * NREG * KCH * NSUB_MAX);
  const uint64_t o_bs = take(4ull * (NBIN_MAX + 1));
  const uint64_t o_bad = take(4ull * HEAD_WG);
  const uint64_t o_bc = take(sizeof(Cand) * n);
  const uint64_t o_np = take(sizeof(NewPair) * n);
  if (ws) {
    char *b = static_cast<char *>(base);
    ws->hdr = reinterpret_cast<WsHdr *>(b + o_hdr);
    ws->pos = reinterpret_cast<uint64_t *>(b + o_pos);
    ws->dd = reinterpret_cast<DSlot *>(b + o_dd);
    ws->trig = reinterpret_cast<uint64_t *>(b + o_trig);
    ws->def = reinterpret_cast<uint64_t *>(b + o_def);
    ws->cand = reinterpret_cast<Cand *>(b + o_cand);
    ws->cand_cnt = reinterpret_cast<uint32_t *>(b + o_cc);
    ws->ctot = reinterpret_cast<uint32_t *>(b + o_ct);
    ws->soff = reinterpret_cast<uint32_t *>(b + o_soff);
    ws->rcnt = reinterpret_cast<uint32_t *>(b + o_rcnt);
    ws->hist2 = reinterpret_cast<uint32_t *>(b + o_h2);
    ws->base2 = reinterpret_cast<uint32_t *>(b + o_b2);
    ws->bstart = reinterpret_cast<uint32_t *>(b + o_bs);
    ws->bad = reinterpret_cast<uint32_t *>(b + o_bad);
    ws->bcand = reinterpret_cast<Cand *>(b + o_bc);
    ws->np = reinterpret_cast<NewPair *>(b + o_np);
    ws->n_dedupe = nd;
    ws->list_cap = nl;
    ws->seg = seg;
  }
  return off;
}

__device__ __forceinline__ void ws_error(WsHdr *h, int e) { atomicCAS(&h->err, 0, e); }

// Returns the dedupe slot when this call created the entry (first sighting of the
// pair), -1 when it was there, -2 on an error (recorded).  TRY: compare-and-swap without a
// look first -- two round trips for a new pair instead of four, where few meet on a slot (one
// of a workgroup, see met_pair); else the look keeps most of them off the atomics.
template <bool TRY>
__device__ int64_t dedupe_pair(const InsWs &ws, uint64_t nd, uint64_t key, uint64_t mine) {
  uint64_t h = mix64(key ^ ((mine >> 32) * 0xC2B2AE3D27D4EB4Full)) & (nd - 1);
  for (uint64_t step = 0; step < nd; ++step, h = (h + 1) & (nd - 1)) {
    DSlot *d = ws.dd + h;
    uint64_t k = TRY ? KEY_EMPTY : __hip_atomic_load(&d->key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (k == KEY_EMPTY) k = atomicCAS(reinterpret_cast<unsigned long long *>(&d->key), KEY_EMPTY, key);
    if (k != KEY_EMPTY && k != key) continue;
    // this slot's key is `key`; its owner instance is decided by the second word
    uint64_t w = TRY ? 0 : __hip_atomic_load(&d->w2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while (true) {
      if (w == 0) {
        const uint64_t prev = atomicCAS(reinterpret_cast<unsigned long long *>(&d->w2), 0ull, mine);
        if (prev == 0) return int64_t(h);
        w = prev;
        continue;
      }
      if ((w >> 32) == (mine >> 32)) {
        if (mine < w) atomicMin(reinterpret_cast<unsigned long long *>(&d->w2), mine);
        return -1;
      }
      break;  // another instance's pair: keep probing
    }
  }
  ws_error(ws.hdr, SMETRIC_EINTERNAL);
  return -2;
}

// The pairs that a workgroup of a find pass has met, each with its lowest request, in LDS: of
// a prefix that many of its requests enter, one pair goes on to the dedupe table.  True: the
// pair was met with a request as low or lower, and whoever met it enters it.  False: new, or to
// be lowered, or no room within a few slots (it then goes on like a new one).
// Atomics on one word of memory take 12 ns each, so 16,384 requests entering 16 blocks
// on one instance (each pair 16,384 times) took 428 us in the probed find pass and 176 in
// the self-contained one, now 19 and 39; 4,096 entering 64 blocks 128 and 252, now 21 and 23.
template <int NT>
struct MetPairs {
  unsigned long long k[2 * NT], w[2 * NT];  // as DSlot
};
template <int NT>
__device__ __forceinline__ void met_clear(MetPairs<NT> &mp) {
  for (int h = threadIdx.x; h < 2 * NT; h += NT) mp.k[h] = mp.w[h] = 0;
  __syncthreads();
}
template <int NT>
__device__ __forceinline__ bool met_pair(MetPairs<NT> &mp, uint64_t key, uint64_t mine) {
  uint32_t h = uint32_t(mix64(key ^ ((mine >> 32) * 0xC2B2AE3D27D4EB4Full)));
  for (int step = 0; step < 4; ++step, ++h) {
    unsigned long long *pk = &mp.k[h % (2 * NT)], *pw = &mp.w[h % (2 * NT)];
    unsigned long long k = *pk;
    if (k == KEY_EMPTY) k = atomicCAS(pk, 0ull, (unsigned long long)key);
    if (k != KEY_EMPTY && k != key) continue;
    unsigned long long w = *pw;
    if (w == 0) w = atomicCAS(pw, 0ull, (unsigned long long)mine);
    if (w == 0) return false;
    if ((w >> 32) != (mine >> 32)) continue;  // another instance's pair
    return w <= mine || atomicMin(pw, (unsigned long long)mine) <= mine;
  }
  return false;
}

// Append `h` (when >= 0) to the list: one atomicAdd per wavefront for all its lanes.
__device__ __forceinline__ void append_wave(unsigned long long *counter, uint64_t *list, uint64_t cap, int64_t h) {
  const uint64_t want = __ballot(h >= 0);
  if (!want) return;
  const int lane = threadIdx.x & 63;
  const int leader = __builtin_ctzll(want);
  unsigned long long base = 0;
  if (lane == leader) base = atomicAdd(counter, (unsigned long long)__popcll(want));
  base = __shfl(base, leader, 64);
  if (h >= 0) {
    const unsigned long long at = base + __popcll(want & ((uint64_t(1) << lane) - 1));
    if (at < cap) list[at] = uint64_t(h);  // more pairs than blocks: rejected by the check
  }
}

__device__ __forceinline__ bool range_of(const int64_t *blk_off, int r, int64_t n_blocks, int64_t &b0,
                                         int64_t &nb) {
  b0 = blk_off[r];
  const int64_t b1 = blk_off[r + 1];
  nb = b1 - b0;
  return b0 >= 0 && b0 <= b1 && b1 <= n_blocks;
}

// One launch clears the workspace's header and the pair table.
__global__ __launch_bounds__(TB) void ins_clear_kernel(InsWs ws) {
  const uint64_t stride = uint64_t(gridDim.x) * TB, t = uint64_t(blockIdx.x) * TB + threadIdx.x;
  if (t < sizeof(WsHdr) / 8) reinterpret_cast<uint64_t *>(ws.hdr)[t] = 0;
  for (uint64_t h = t; h < ws.n_dedupe; h += stride) ws.dd[h] = DSlot{0, 0};
}

// What the find pass leaves per block in pos: nothing, the slot + 1 of an entry to refresh,
// or POS_NEW | the pair-table slot of a new pair that this block entered first.
constexpr uint64_t POS_NEW = uint64_t(1) << 63;

// Grid of the find and apply passes: one atomic per workgroup on the pass's counter (12 ns
// each when they meet on one word), so few and large workgroups where there are many blocks.
inline int find_threads(uint64_t threads) { return threads <= uint64_t(FIND_WG) * TB ? TB : 4 * TB; }
inline int find_grid(uint64_t threads) {
  const uint64_t nt = find_threads(threads), g = (threads + nt - 1) / nt;
  return int(g < 1 ? 1 : (g > 2 * FIND_WG ? 2 * FIND_WG : g));
}

// Waits until this wavefront's memory operations have completed.
__device__ __forceinline__ void memory_done() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
}

// End of a find pass.  The last workgroup to get here makes the all-or-nothing check -- the
// first input error, or EFULL, leaves the index unchanged -- so the check costs no launch of
// its own: every workgroup adds, in one atomic, its turn, whether it met an error, and its
// new pairs, and the one whose turn is the last has the totals in the returned word.  The
// words that pass between workgroups are all accessed by atomics, and a workgroup's are
// complete before its turn, so no cache is written back.  This rests on the hardware (an
// atomic of device scope acts in one place for all dies, and one that has been waited for has
// acted), not on the memory model, whose release and acquire here cost 5 us of cache
// write-back.  n_entries: as read when the kernel began (nothing else changes it meanwhile).
constexpr int TURN_SHIFT = 40, ERR_SHIFT = 52;  // 2^40 new pairs, 2^12 workgroups
static_assert(2 * FIND_WG < (1 << 12) && DEDUPE_WG < (1 << 12), "turns and errors fit their fields");
template <bool PAIRS>
__device__ void ins_check_last(const DevIndex &ix, const InsWs &ws, int64_t n_blocks, unsigned long long n_entries,
                               uint32_t n_new, uint64_t n_pairs, bool bad) {
  __shared__ unsigned long long s_new, s_pairs;
  __shared__ bool s_bad;
  if (threadIdx.x == 0) {
    s_new = s_pairs = 0;
    s_bad = false;
  }
  memory_done();  // every wavefront's error code has reached the device's coherence point
  __syncthreads();
  if (n_new) atomicAdd(&s_new, (unsigned long long)n_new);
  if (PAIRS && n_pairs) atomicAdd(&s_pairs, (unsigned long long)n_pairs);
  if (bad) s_bad = true;
  __syncthreads();
  if (threadIdx.x != 0) return;
  WsHdr *h = ws.hdr;
  if (PAIRS && s_pairs) {
    atomicAdd(&h->n_pairs, s_pairs);
    memory_done();
  }
  const unsigned long long mine = s_new + (1ull << TURN_SHIFT) + (s_bad ? 1ull << ERR_SHIFT : 0ull);
  const unsigned long long all = atomicAdd(&h->turns, mine) + mine;
  if (((all >> TURN_SHIFT) & ((1u << (ERR_SHIFT - TURN_SHIFT)) - 1)) != gridDim.x) return;
  const unsigned long long total = all & ((1ull << TURN_SHIFT) - 1);
  int e = 0;
  if (all >> ERR_SHIFT) e = __hip_atomic_load(&h->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else if (PAIRS && __hip_atomic_load(&h->n_pairs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >
                        (unsigned long long)n_blocks)
    e = SMETRIC_EINVAL;
  if (e == 0 && n_entries + total > ix.capacity) e = SMETRIC_EFULL;
  if (e != 0) {
    h->abort = 1;
    set_status(ix.hdr, e);
  } else {
    ix.hdr->n_entries = n_entries + total;
  }
}

// Find and dedupe, self-contained: groups of `per` threads (a wavefront or TB threads) take
// requests, their threads blocks.
template <int NT>
__global__ __launch_bounds__(NT) void ins_probe_kernel(DevIndex ix, InsWs ws, const uint64_t *keys,
                                                       const int64_t *blk_off, int32_t n_req, int64_t n_blocks,
                                                       const int32_t *instance, const uint32_t *session,
                                                       uint32_t epoch, int per) {
  __shared__ MetPairs<NT> met;
  met_clear(met);
  const int gt = threadIdx.x % per, groups = NT / per;
  const unsigned long long n_entries = ix.hdr->n_entries;
  uint64_t pairs = 0;
  uint32_t n_new = 0;
  bool bad = false;
  for (int64_t r = int64_t(blockIdx.x) * groups + threadIdx.x / per; r < n_req; r += int64_t(gridDim.x) * groups) {
    int64_t b0, nb;
    if (!range_of(blk_off, int(r), n_blocks, b0, nb)) {
      bad = true;
      continue;
    }
    if (nb == 0) continue;
    if (gt == 0) pairs += uint64_t(nb);
    const int32_t inst = instance[r];
    const uint32_t sess = session[r];
    if (inst < 0 || inst >= ix.n_inst || sess >= SESSION_LIMIT) {
      bad = true;
      continue;
    }
    for (int64_t j = gt; j < nb; j += per) {
      const uint64_t key = keys[b0 + j];
      uint64_t at = 0;
      if (key == KEY_EMPTY || key == KEY_TOMB) {
        bad = true;
      } else {
        const Found f = find_entry(ix, key, uint32_t(inst));
        if (f.slot >= 0) {
          at = val_epoch(f.val) < epoch ? uint64_t(f.slot) + 1 : 0;
        } else if (const uint64_t w2 = ((uint64_t(inst) + 1) << 32) | uint32_t(r); !met_pair(met, key, w2)) {
          const int64_t h = dedupe_pair<true>(ws, ws.n_dedupe, key, w2);
          at = h >= 0 ? POS_NEW | uint64_t(h) : 0;
          n_new += h >= 0;
          bad |= h == -2;
        }
      }
      ws.pos[b0 + j] = at;
    }
  }
  if (bad) ws_error(ws.hdr, SMETRIC_EINVAL);
  ins_check_last<true>(ix, ws, n_blocks, n_entries, n_new, pairs, bad);
}

// The same from the direct form of a probe state: threads take blocks, and the descriptor
// answers for blocks of no or one holder.
template <int NT>
__global__ __launch_bounds__(NT) void insd_find_kernel(DevIndex ix, ProbeView pv, InsWs ws, int64_t n_blocks,
                                                       const int32_t *instance, const uint32_t *session,
                                                       uint32_t epoch) {
  __shared__ MetPairs<NT> met;
  met_clear(met);
  const unsigned long long n_entries = ix.hdr->n_entries;
  bool bad = pv.hdr->err != 0;
  const int64_t n = bad ? 0 : n_blocks;
  uint32_t n_new = 0;
  for (int64_t p = int64_t(blockIdx.x) * NT + threadIdx.x; p < n; p += int64_t(gridDim.x) * NT) {
    const uint64_t key = pv.part_key[p], d = pv.desc_p[p];
    const uint32_t r = pv.part_req[p];
    const int32_t inst = instance[r];
    uint64_t at = 0;
    if (inst < 0 || inst >= ix.n_inst || session[r] >= SESSION_LIMIT || key == KEY_EMPTY || key == KEY_TOMB) {
      bad = true;
    } else {
      const uint32_t kind = desc_kind(d);
      int64_t slot = -1;
      bool raise = true;
      if (kind == D_ONE) {
        if (desc_inst(d) == uint32_t(inst)) slot = int64_t(desc_x(d));
      } else if (kind == D_HOT || kind == D_MANY) {
        const Found f = kind == D_HOT ? find_holder(ix, desc_x(d), key, uint32_t(inst)) : find_entry(ix, key, uint32_t(inst));
        slot = f.slot;
        raise = val_epoch(f.val) < epoch;
      }
      if (slot >= 0) {
        at = raise ? uint64_t(slot) + 1 : 0;
      } else if (const uint64_t w2 = ((uint64_t(inst) + 1) << 32) | r; !met_pair(met, key, w2)) {
        const int64_t h = dedupe_pair<true>(ws, ws.n_dedupe, key, w2);
        at = h >= 0 ? POS_NEW | uint64_t(h) : 0;
        n_new += h >= 0;
        bad |= h == -2;
      }
    }
    ws.pos[p] = at;
  }
  if (bad) ws_error(ws.hdr, SMETRIC_EINVAL);
  ins_check_last<false>(ix, ws, n_blocks, n_entries, n_new, 0, bad);
}

// What the find pass left for one block.  A refreshed entry's value is read first, so an
// entry that many requests share is raised by few of them; new pairs claim EMPTY slots
// only, so the two never touch one value except an entry that both raise to one epoch.
__device__ __forceinline__ void apply_pos(const DevIndex &ix, const InsWs &ws, uint64_t at, const uint32_t *session,
                                          uint32_t epoch) {
  int64_t tk = -1, df = -1;
  bool rf = false;
  if (at & POS_NEW) {
    const int64_t h = int64_t(at & ~POS_NEW);
    const DSlot d = ws.dd[h];
    bool trig;
    const int pl = place_new(ix, d.key, dd_inst(d.w2), epoch, session[dd_req(d.w2)], trig, true);
    if (pl == FAILED) set_status(ix.hdr, SMETRIC_EINTERNAL);
    else if (pl == DEFERRED) df = h;
    else if (pl == REFRESHED) rf = true;  // a block past its probe bound that was an entry
    else if (trig) tk = h;
  } else if (at) {
    uint64_t *vp = val_ptr(ix, int64_t(at - 1));
    const uint64_t v = *vp;
    if (val_epoch(v) < epoch) set_epoch_at(vp, val_kind(v), val_inst(v), epoch);
  }
  uncount_refreshed(ix, rf);
  append_wave(&ws.hdr->n_trig, ws.trig, ws.list_cap, tk);  // by pair-table slot
  append_wave(&ws.hdr->n_def, ws.def, ws.list_cap, df);
}

// Apply; blk_off null: the blocks of a direct probe state, else those of every request.
template <int NT>
__global__ __launch_bounds__(NT) void ins_apply_kernel(DevIndex ix, InsWs ws, const int64_t *blk_off, int32_t n_req,
                                                       int64_t n_blocks, const uint32_t *session, uint32_t epoch,
                                                       int per) {
  if (ws.hdr->abort) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) keep_epoch_top(ix, epoch);
  const int lane = threadIdx.x & 63;
  if (blk_off) {
    const int groups = NT / per;
    for (int64_t r = int64_t(blockIdx.x) * groups + threadIdx.x / per; r < n_req; r += int64_t(gridDim.x) * groups) {
      int64_t b0, nb;
      if (!range_of(blk_off, int(r), n_blocks, b0, nb)) continue;
      for (int64_t j0 = (threadIdx.x % per) & ~63; j0 < nb; j0 += per)  // whole wavefronts iterate together
        apply_pos(ix, ws, j0 + lane < nb ? ws.pos[b0 + j0 + lane] : 0, session, epoch);
    }
  } else {
    for (int64_t p0 = int64_t(blockIdx.x) * NT + (threadIdx.x & ~63); p0 < n_blocks; p0 += int64_t(gridDim.x) * NT)
      apply_pos(ix, ws, p0 + lane < n_blocks ? ws.pos[p0 + lane] : 0, session, epoch);
  }
}

// Convert the queued keys.  trig holds indexes: key = np[idx].key when `np` is given
// (region-ordered insert: new-pair positions), dd[idx].key when `dd` is (insert: pair-table
// slots), else keys[idx] (rebuild).
__global__ void spill_kernel(DevIndex ix, const uint64_t *trig, const unsigned long long *n_trig,
                             const int *abort_flag, const uint64_t *keys, const DSlot *dd, const NewPair *np) {
  if (abort_flag && *abort_flag) return;
  const uint64_t n = *n_trig;
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
    const uint64_t t = trig[i];
    const uint64_t key = np ? np[t].key : (dd ? dd[t].key : keys[t]);
    if (!spill_key(ix, key)) set_status(ix.hdr, SMETRIC_EINTERNAL);
  }
}

// ---------------------------------------------------------------------------------
// Region-ordered insert, from the descriptors of smetric_probe
// ---------------------------------------------------------------------------------
// Pipeline (no sort, no global atomics on the way to the distinct new pairs), nine launches
// (thirteen before the clear took the request checks, the count the sizing, the scatter the
// fallback table's clear and the dedupe the check: 4.6 us each behind busy kernels; batches of
// 1 to 5 M blocks 13 us faster each):
//   classify   per block in region order: refresh position, or candidate appended to the
//              region's part of the workgroup's segment; when no error can abort the
//              insert (checked beforehand: keys, requests, capacity for every block) the
//              refresh is done here and its pass is skipped
//   bins       the candidates partitioned into NREG x nsub bins of home buckets (count,
//              scan, scatter, as the probe's region partition), so all candidates of a
//              pair share a bin
//   dedupe     one workgroup per bin: an LDS pair table keeps each (key, instance) once
//              with its lowest request; bins above BIN_CAP stream through it, and one whose
//              distinct pairs would fill it uses the global pair table
//              The last workgroup checks all-or-nothing: EINVAL or EFULL leave the index
//              unchanged
//   refresh    epoch = max(old, epoch) at the classified positions (if not done above)
//   place      distinct new pairs in bin (so region) order; spill and deferred as above
// find_member with each bucket read whole (keys and values in one 128-byte request), so
// a chain step is one round trip.
__device__ Found find_member_line(const DevIndex &ix, uint64_t key, uint32_t inst) {
  ChainWalk cw = chain_start(member_bucket(key, inst, ix.n_buckets, ix.nb_inv), member_cls(key, inst));
  bool had_empty;
  do {
    const uint64_t m = cw.b;
    const ulonglong2 *p = reinterpret_cast<const ulonglong2 *>(ix.slots + m * BUCKET_WORDS);
    ulonglong2 kk[SLOTS / 2], vv[SLOTS / 2];
#pragma unroll
    for (int i = 0; i < SLOTS / 2; ++i) kk[i] = p[i];
#pragma unroll
    for (int i = 0; i < SLOTS / 2; ++i) vv[i] = p[SLOTS / 2 + i];
    bool end = false;
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      const uint64_t k = (s & 1) ? kk[s / 2].y : kk[s / 2].x;
      const uint64_t v = (s & 1) ? vv[s / 2].y : vv[s / 2].x;
      end |= k == KEY_EMPTY;
      if (!end && k == key && val_kind(v) == MEMBER && val_inst(v) == inst) return Found{int64_t(m * SLOTS + s), v};
    }
    had_empty = end;
  } while (chain_next(ix, cw, had_empty));
  return Found{-1, 0};
}

// classify: per probed block (region order), is (key, target) already an entry?  The
// descriptor answers it for NONE and ONE; HOT needs the bitmap bit and the member slot
// (inside the key's region), MANY a chain walk.  Existing -> refresh position; absent ->
// candidate, appended to the part of this workgroup's segment that holds its region
// (LDS counters, no global atomics).  The part of region g has room for every position
// of the workgroup in g: with F(x) = the workgroup's positions below x, it starts at
// F(start of g).
// All INS_WG workgroups advance through the region order together.  Each thread takes
// CU positions per round (the same positions as a plain grid-stride loop, so segments
// keep their bound), with every load of the round issued before any result is used.
__device__ __forceinline__ uint32_t positions_below(uint64_t x, uint64_t span, uint32_t w) {
  const uint64_t r = x % span, lo = uint64_t(w) * TB;
  return uint32_t((x / span) * TB + (r <= lo ? 0 : (r - lo < TB ? r - lo : TB)));
}

__global__ __launch_bounds__(TB) void insp_classify_kernel(DevIndex ix, ProbeView pv, InsWs ws,
                                                           const int32_t *instance, const uint32_t *session,
                                                           uint32_t epoch) {
  __shared__ unsigned int lc[NREG];
  __shared__ uint32_t part[NREG];
  __shared__ unsigned long long rb[NREG + 1];  // region boundaries in position order
  const int tid = threadIdx.x;
  const uint64_t span = uint64_t(gridDim.x) * TB;
  if (tid == 0) {
    unsigned long long acc = 0;
    for (int g = 0; g < NREG; ++g) {
      rb[g] = acc;
      acc += pv.hdr->tot[g];
    }
    rb[NREG] = acc;
  }
  __syncthreads();
  if (tid < NREG) {
    lc[tid] = 0;
    part[tid] = positions_below(rb[tid], span, blockIdx.x);
  }
  __syncthreads();
  const uint64_t n = pv.hdr->n;
  if (pv.hdr->err) {
    if (blockIdx.x == 0 && tid == 0) ws_error(ws.hdr, SMETRIC_EINVAL);
    if (tid < NREG) {
      ws.rcnt[uint64_t(blockIdx.x) * NREG + tid] = 0;
      ws.soff[uint64_t(blockIdx.x) * NREG + tid] = 0;
    }
    if (tid == 0) ws.cand_cnt[blockIdx.x] = 0;
    return;
  }
  // No error can abort this insert (valid keys and requests; even if every block were a new
  // entry the index would not overflow): refreshes are done here, in place.
  const bool req_bad = __ballot(ws.bad[tid & (HEAD_WG - 1)] != 0) != 0;  // one flag per lane
  const bool inl = !pv.hdr->bad_key && !req_bad && ix.hdr->n_entries + n <= ix.capacity;
  const bool top = epoch_tops(ix, epoch);
  if (blockIdx.x == 0 && tid == 0) ws.hdr->inl = inl;
  Cand *seg = ws.cand + uint64_t(blockIdx.x) * ws.seg;
  constexpr int CU = 2;
  int gcur = 0;  // region of this thread's current position (positions only increase)
  for (uint64_t i0 = uint64_t(blockIdx.x) * TB + tid; i0 < n; i0 += CU * span) {
    // positions past the end read the last position (in bounds) and are dropped below
    uint64_t key[CU], d[CU];
    uint32_t r[CU];
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      const uint64_t i = i0 + u * span < n ? i0 + u * span : n - 1;
      key[u] = pv.part_key[i];
      r[u] = pv.part_req[i];
      d[u] = pv.desc_p[i];
    }
    int32_t t[CU];
    uint32_t sess[CU];
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      t[u] = instance[r[u]];
      sess[u] = session[r[u]];
    }
    // HOT: the target's bitmap word (a block of another kind reads record 0, always present)
    uint64_t hw[CU];
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      const bool hot = desc_kind(d[u]) == D_HOT && t[u] >= 0 && t[u] < ix.n_inst;
      hw[u] = ix.pool[(hot ? desc_x(d[u]) : 0) * uint64_t(ix.words) + (hot ? uint32_t(t[u]) >> 6 : 0u)];
    }
    int64_t slot[CU];
    bool fresh[CU];
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      slot[u] = -1;
      fresh[u] = false;
      const uint64_t i = i0 + u * span;
      if (i >= n) continue;
      while (gcur < NREG - 1 && rb[gcur + 1] <= i) ++gcur;
      if (t[u] < 0 || t[u] >= ix.n_inst || sess[u] >= SESSION_LIMIT || key[u] == KEY_EMPTY || key[u] == KEY_TOMB) {
        ws_error(ws.hdr, SMETRIC_EINVAL);
      } else {
        const uint32_t kind = desc_kind(d[u]);
        if (kind == D_ONE) {
          if (desc_inst(d[u]) == uint32_t(t[u])) slot[u] = int64_t(desc_x(d[u]));
        } else if (kind == D_HOT) {
          if ((hw[u] >> (t[u] & 63)) & 1) {
            const Found f = find_member_line(ix, key[u], uint32_t(t[u]));
            slot[u] = f.slot;
            fresh[u] = val_epoch(f.val) >= epoch;
          }
        } else if (kind == D_MANY) {
          const Found f = find_entry(ix, key[u], uint32_t(t[u]));
          slot[u] = f.slot;
          fresh[u] = val_epoch(f.val) >= epoch;
        }
        if (slot[u] < 0)
          seg[part[gcur] + atomicAdd(&lc[gcur], 1u)] = Cand{key[u], ((uint64_t(t[u]) + 1) << 32) | r[u]};
      }
    }
    if (inl) {
      // epoch = max(old, epoch) without a read: the entry is (key, t), a member for a HOT
      // key and a plain slot otherwise.  A store while no entry can be above the epoch: 21M
      // refreshes in a table of 4.3 GB, this kernel 980 -> 790 us per batch; 3.1M in one of
      // some 150 MB, 161 -> 68 us.  Where the slot was found by a walk its value is already
      // here, and an entry seen at the epoch (or a newer one) is left alone: a shared prefix's
      // members are refreshed by every request routed to their instance, and atomics on one
      // address are served one after another (8,192 requests sharing 2,048 blocks on 128
      // instances, with atomics: 7.1 -> 1.0 ms per batch).
#pragma unroll
      for (int u = 0; u < CU; ++u)
        if (slot[u] >= 0 && !fresh[u]) {
          uint64_t *vp = val_ptr(ix, slot[u]);
          const uint32_t kind = desc_kind(d[u]) == D_HOT ? MEMBER : PLAIN;
          if (top) set_epoch_at(vp, kind, uint32_t(t[u]), epoch);
          else raise_epoch_at(vp, kind, uint32_t(t[u]), epoch);
        }
    } else {
#pragma unroll
      for (int u = 0; u < CU; ++u)
        if (i0 + u * span < n) ws.pos[i0 + u * span] = slot[u] >= 0 ? uint64_t(slot[u]) + 1 : 0;
    }
  }
  __syncthreads();
  if (tid < NREG) {
    ws.rcnt[uint64_t(blockIdx.x) * NREG + tid] = lc[tid];
    ws.soff[uint64_t(blockIdx.x) * NREG + tid] = part[tid];
  }
  if (tid == 0) {
    unsigned int all = 0;
    for (int g = 0; g < NREG; ++g) all += lc[g];
    ws.cand_cnt[blockIdx.x] = all;
  }
}

// Clears the workspace's header and flags requests whose target or session is out of range
// (the classify pass then takes the path that checks every block before the index changes):
// each of HEAD_WG workgroups leaves its own flag, so nothing has to be cleared before.
__global__ __launch_bounds__(TB) void insp_head_kernel(DevIndex ix, InsWs ws, const int32_t *instance,
                                                       const uint32_t *session, int32_t n_req) {
  if (blockIdx.x == 0 && threadIdx.x < sizeof(WsHdr) / 8) reinterpret_cast<uint64_t *>(ws.hdr)[threadIdx.x] = 0;
  int bad = 0;
  for (int32_t r = blockIdx.x * TB + threadIdx.x; r < n_req; r += gridDim.x * TB)
    bad |= instance[r] < 0 || instance[r] >= ix.n_inst || session[r] >= SESSION_LIMIT;
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) ws.bad[blockIdx.x] = uint32_t(bad);
}

// Sum of n 32-bit counts, by one workgroup of TB threads (eight loads in flight per thread).
__device__ unsigned long long sum_counts(const uint32_t *cnt, uint32_t n) {
  __shared__ unsigned long long part[TB / 64];
  unsigned long long c = 0;
  for (uint32_t w0 = 0; w0 < n; w0 += 8 * TB) {
    uint32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t w = w0 + u * TB + threadIdx.x;
      v[u] = w < n ? cnt[w] : 0u;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) c += v[u];
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
  __syncthreads();
  unsigned long long all = 0;
#pragma unroll
  for (int i = 0; i < TB / 64; ++i) all += part[i];
  __syncthreads();
  return all;
}

// total candidates -> bins per region: the least power of two that keeps the mean bin at
// or below BIN_TARGET candidates (at most NSUB_MAX)
__device__ __forceinline__ uint32_t bins_per_region(unsigned long long n_cand) {
  uint32_t nsub = 1;
  while (nsub < uint32_t(NSUB_MAX) && uint64_t(nsub) * NREG * BIN_TARGET < n_cand) nsub <<= 1;
  return nsub;
}

// Bin of a key among NREG * nsub equal ranges of home buckets; bin / nsub is its region.
__device__ __forceinline__ uint32_t bin_of(uint64_t key, uint64_t n_buckets, uint64_t nb_inv, uint32_t nsub) {
  return uint32_t(scaled_floor(home_bucket(key, n_buckets), uint64_t(NREG) * nsub, n_buckets, nb_inv));
}

// The candidates of chunk (g, c): the region-g parts of classify segments
// [c SEG_PER_CH, (c + 1) SEG_PER_CH), seen as one array through the parts' prefix sums.
struct ChunkParts {
  uint32_t pre[SEG_PER_CH + 1];  // prefix of the parts' counts
  uint64_t at[SEG_PER_CH];       // start of each part in ws.cand
};
__device__ void chunk_parts(const InsWs &ws, int g, int c, ChunkParts &cp) {
  if (threadIdx.x == 0) {
    uint32_t acc = 0;
    for (int p = 0; p < SEG_PER_CH; ++p) {
      const uint64_t w = uint64_t(c) * SEG_PER_CH + p;
      cp.pre[p] = acc;
      cp.at[p] = w * ws.seg + ws.soff[w * NREG + g];
      acc += ws.rcnt[w * NREG + g];
    }
    cp.pre[SEG_PER_CH] = acc;
  }
  __syncthreads();
}
__device__ __forceinline__ const Cand *chunk_item(const InsWs &ws, const ChunkParts &cp, uint32_t v) {
  int lo = 0, hi = SEG_PER_CH;  // the part p with pre[p] <= v < pre[p + 1]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cp.pre[mid] <= v) lo = mid;
    else hi = mid;
  }
  return ws.cand + cp.at[lo] + (v - cp.pre[lo]);
}

// Count pass of the bin partition: every workgroup sizes the bins from the segments' counts
// (4 KB each, cheaper than a launch), then workgroup (g, c) histograms its chunk over region g's
// bins (eight candidates per thread per round, loads first) and records the chunk's size.
__global__ __launch_bounds__(TB) void insp_bcount_kernel(DevIndex ix, InsWs ws) {
  __shared__ ChunkParts cp;
  __shared__ uint32_t h[NSUB_MAX];
  const int g = blockIdx.x / KCH, c = blockIdx.x % KCH;
  const unsigned long long n_cand = sum_counts(ws.cand_cnt, INS_WG);
  const uint32_t nsub = bins_per_region(n_cand);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ws.hdr->n_cand = n_cand;
    ws.hdr->nsub = nsub;
  }
  for (int s = threadIdx.x; s < NSUB_MAX; s += TB) h[s] = 0;
  chunk_parts(ws, g, c, cp);  // synchronises
  const uint32_t m = cp.pre[SEG_PER_CH];
  constexpr int UC = 8;
  for (uint32_t v0 = 0; v0 < m; v0 += UC * TB) {
    uint64_t k[UC];
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      const uint32_t v = v0 + u * TB + threadIdx.x;
      k[u] = v < m ? chunk_item(ws, cp, v)->key : 0;
    }
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      if (v0 + u * TB + threadIdx.x < m) {
        const uint32_t sub = bin_of(k[u], ix.n_buckets, ix.nb_inv, nsub) - uint32_t(g) * nsub;
        atomicAdd(&h[sub < nsub ? sub : nsub - 1], 1u);
      }
    }
  }
  __syncthreads();
  uint32_t *out = ws.hist2 + (uint64_t(g) * KCH + c) * NSUB_MAX;
  for (uint32_t s = threadIdx.x; s < nsub; s += TB) out[s] = h[s];
  if (threadIdx.x == 0) ws.ctot[g * KCH + c] = m;
}

// Scan pass: workgroup g gives every bin of region g its first position (regions in
// order, bins in order inside a region) and every (chunk, bin) its running offset; bins
// larger than BIN_CAP add their size to n_over.  One thread per bin, its KCH chunk
// counts loaded at once.
constexpr int SCAN_T = NSUB_MAX;
static_assert(NREG * KCH <= SCAN_T, "one chunk total per thread for the region start");
__global__ __launch_bounds__(SCAN_T) void insp_bscan_kernel(InsWs ws) {
  __shared__ uint32_t wt[SCAN_T / 64];
  __shared__ unsigned long long red[SCAN_T / 64];
  const int g = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint32_t nsub = uint32_t(ws.hdr->nsub);
  // first position of region g: the chunks of every region before it
  unsigned long long before = t < g * KCH ? ws.ctot[t] : 0u;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) before += __shfl_xor(before, d, 64);
  if (lane == 0) red[wave] = before;
  const uint32_t *hg = ws.hist2 + uint64_t(g) * KCH * NSUB_MAX + t;
  uint32_t hc[KCH];
#pragma unroll
  for (int c = 0; c < KCH; ++c) hc[c] = uint32_t(t) < nsub ? hg[uint64_t(c) * NSUB_MAX] : 0u;
  uint32_t tot = 0;
#pragma unroll
  for (int c = 0; c < KCH; ++c) tot += hc[c];
  uint32_t x = tot;  // inclusive scan of the bin totals over the workgroup
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) wt[wave] = x;
  __syncthreads();
  unsigned long long start = 0;
#pragma unroll
  for (int i = 0; i < SCAN_T / 64; ++i) start += red[i];
  uint32_t pre = x - tot;
  for (int i = 0; i < wave; ++i) pre += wt[i];
  if (uint32_t(t) < nsub) {
    const uint32_t first = uint32_t(start) + pre;
    ws.bstart[uint64_t(g) * nsub + t] = first;
    uint32_t acc = first;
    uint32_t *bg = ws.base2 + uint64_t(g) * KCH * NSUB_MAX + t;
#pragma unroll
    for (int c = 0; c < KCH; ++c) {
      bg[uint64_t(c) * NSUB_MAX] = acc;
      acc += hc[c];
    }
    if (tot > uint32_t(BIN_CAP)) atomicAdd(&ws.hdr->n_over, (unsigned long long)tot);
    if (g == NREG - 1 && uint32_t(t) == nsub - 1) ws.bstart[uint64_t(NREG) * nsub] = acc;
  }
}

// Scatter pass: workgroup (g, c) moves its chunk into bin order one tile at a time (LDS
// ranks per bin, the tile regrouped by bin in LDS, each bin's part written as one run
// after the previous tile's).  The workgroups also size and clear the fallback pair table for
// the pass after this one: a power of two >= 2 x the candidates of all bins above BIN_CAP,
// though most of those never need it (what they need shows only there).
constexpr int U2 = 8;
constexpr int TILE2 = U2 * TB;
static_assert(NSUB_MAX % TB == 0, "bins per thread in the scans");
__global__ __launch_bounds__(TB) void insp_bscatter_kernel(DevIndex ix, InsWs ws) {
  __shared__ ChunkParts cp;
  __shared__ uint32_t cnt[NSUB_MAX], tstart[NSUB_MAX], run[NSUB_MAX], wt[TB / 64];
  __shared__ Cand sc[TILE2];
  __shared__ uint16_t ssub[TILE2];
  const int g = blockIdx.x / KCH, c = blockIdx.x % KCH, t = threadIdx.x;
  const uint32_t nsub = uint32_t(ws.hdr->nsub);
  if (const unsigned long long over = ws.hdr->n_over) {
    uint64_t nd = 64;
    while (nd < 2 * over && nd < ws.n_dedupe) nd <<= 1;
    if (blockIdx.x == 0 && t == 0) ws.hdr->n_dd2 = nd;
    for (uint64_t h = uint64_t(blockIdx.x) * TB + t; h < nd; h += uint64_t(gridDim.x) * TB) ws.dd[h] = DSlot{0, 0};
  }
  const uint32_t *b2 = ws.base2 + (uint64_t(g) * KCH + c) * NSUB_MAX;
  for (uint32_t s = t; s < NSUB_MAX; s += TB) {
    run[s] = s < nsub ? b2[s] : 0;
    cnt[s] = 0;
  }
  chunk_parts(ws, g, c, cp);  // synchronises
  const uint32_t m = cp.pre[SEG_PER_CH];
  for (uint32_t t0 = 0; t0 < m; t0 += TILE2) {
    Cand e[U2];
    uint32_t sub[U2], rk[U2];
#pragma unroll
    for (int u = 0; u < U2; ++u) {
      const uint32_t v = t0 + u * TB + t;
      e[u] = v < m ? *chunk_item(ws, cp, v) : Cand{0, 0};
    }
#pragma unroll
    for (int u = 0; u < U2; ++u) {
      const uint32_t s = bin_of(e[u].key, ix.n_buckets, ix.nb_inv, nsub) - uint32_t(g) * nsub;
      sub[u] = s < nsub ? s : nsub - 1;
      rk[u] = t0 + u * TB + t < m ? atomicAdd(&cnt[sub[u]], 1u) : 0;
    }
    __syncthreads();
    // exclusive scan of the tile's bin counts
    constexpr int Q = NSUB_MAX / TB;
    uint32_t q[Q], sum = 0;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      q[j] = cnt[t * Q + j];
      sum += q[j];
    }
    uint32_t x = sum;
    const int lane = t & 63, wave = t >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63) wt[wave] = x;
    __syncthreads();
    uint32_t pre = x - sum;
    for (int i = 0; i < wave; ++i) pre += wt[i];
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      tstart[t * Q + j] = pre;
      pre += q[j];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U2; ++u) {
      if (t0 + u * TB + t < m) {
        const uint32_t p = tstart[sub[u]] + rk[u];
        sc[p] = e[u];
        ssub[p] = uint16_t(sub[u]);
      }
    }
    __syncthreads();
    const uint32_t in_tile = m - t0 < uint32_t(TILE2) ? m - t0 : uint32_t(TILE2);
#pragma unroll
    for (int u = 0; u < U2; ++u) {
      const uint32_t p = u * TB + t;
      if (p < in_tile) {
        const uint32_t s = ssub[p];
        ws.bcand[run[s] + (p - tstart[s])] = sc[p];
      }
    }
    __syncthreads();
    for (uint32_t s = t; s < nsub; s += TB) {
      run[s] += cnt[s];
      cnt[s] = 0;
    }
    __syncthreads();
  }
}

// Enter candidate (key, mine) in a bin's LDS pair table (the pair table's rule: a slot's
// key is claimed first, then its instance; the same pair keeps the lowest request).  True:
// the pair is new there.
__device__ __forceinline__ bool lds_pair(unsigned long long *tk, unsigned long long *tw, uint64_t key,
                                         uint64_t mine) {
  uint32_t h = uint32_t(mix64(key ^ ((mine >> 32) * 0xC2B2AE3D27D4EB4Full))) & (DT - 1);
  for (int step = 0; step < DT; ++step, h = (h + 1) & (DT - 1)) {
    unsigned long long k = tk[h];
    if (k == KEY_EMPTY) k = atomicCAS(&tk[h], 0ull, (unsigned long long)key);
    if (k != KEY_EMPTY && k != key) continue;
    unsigned long long w = tw[h];
    while (true) {
      if (w == 0) {
        const unsigned long long prev = atomicCAS(&tw[h], 0ull, (unsigned long long)mine);
        if (prev == 0) return true;
        w = prev;
        continue;
      }
      if ((w >> 32) == (mine >> 32)) {
        if (mine < w) atomicMin(&tw[h], (unsigned long long)mine);
        return false;
      }
      break;  // another instance's pair: keep probing
    }
  }
  return false;
}

// Dedupe pass: each bin of at most BIN_CAP candidates is deduplicated in an LDS pair
// table and its distinct pairs written to the front of its range of np (the rest get
// KEY_EMPTY).  A larger bin is mostly one key's pairs over and over (a prefix that many
// requests of the batch share): its candidates stream through the same table, DD_S a thread
// at a time, as long as the distinct pairs leave the table at most half full before each
// round; a bin of more goes through the fallback pair table in place, from its start.
// (8,192 requests sharing 2,048 blocks, four batches in all: 14.0 -> 12.9 ms.)  Workgroups take bins in order; a bin's candidates are loaded (all at once)
// before its table is cleared.
constexpr int DD_T = 512;
constexpr int DD_U = BIN_CAP / DD_T;
constexpr int DD_S = 2;
static_assert(BIN_CAP % DD_T == 0 && DT % DD_T == 0, "whole candidates and slots per thread");
static_assert(DT / 2 + DD_S * DD_T < DT, "a round's new pairs never fill the table");
__global__ __launch_bounds__(DD_T) void insp_bdedupe_kernel(DevIndex ix, InsWs ws) {
  __shared__ unsigned long long tk[DT], tw[DT];
  __shared__ uint32_t wt[DD_T / 64];
  __shared__ uint32_t n_occ;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint32_t nbin = uint32_t(ws.hdr->nsub) * NREG;
  const uint64_t nd2 = ws.hdr->n_dd2;
  const unsigned long long n_entries = ix.hdr->n_entries;
  uint32_t n_new = 0;  // this thread's share of the workgroup's distinct new pairs
  bool bad = t == 0 && blockIdx.x == 0 && ws.hdr->err != 0;  // an error the classify pass met
  for (uint32_t b = blockIdx.x; b < nbin; b += gridDim.x) {
    const uint32_t lo = ws.bstart[b], hi = ws.bstart[b + 1], m = hi - lo;
    if (m == 0) continue;
    const bool big = m > uint32_t(BIN_CAP);
    bool over = false;
    if (big) {
      for (int j = t; j < DT; j += DD_T) {
        tk[j] = 0;
        tw[j] = 0;
      }
      if (t == 0) n_occ = 0;
      __syncthreads();
      for (uint32_t k0 = lo; k0 < hi && !over; k0 += DD_S * DD_T) {  // whole workgroups iterate together
        Cand e[DD_S];
#pragma unroll
        for (int u = 0; u < DD_S; ++u) {
          const uint32_t k = k0 + u * DD_T + t;
          e[u] = k < hi ? ws.bcand[k] : Cand{KEY_EMPTY, 0};
        }
        uint32_t claimed = 0;
#pragma unroll
        for (int u = 0; u < DD_S; ++u)
          if (e[u].key != KEY_EMPTY) claimed += lds_pair(tk, tw, e[u].key, e[u].w2);
        if (claimed) atomicAdd(&n_occ, claimed);
        __syncthreads();
        over = n_occ > uint32_t(DT / 2) && hi - k0 > uint32_t(DD_S * DD_T);
        __syncthreads();  // read by all before the next round adds
      }
    }
    if (over) {
      for (uint32_t k = lo + t; k < hi; k += DD_T) {
        const Cand e = ws.bcand[k];
        const int64_t h = dedupe_pair<false>(ws, nd2, e.key, e.w2);
        ws.np[k] = h >= 0 ? NewPair{e.key, NP_FALLBACK | uint64_t(h)} : NewPair{KEY_EMPTY, 0};
        n_new += h >= 0;
        bad |= h == -2;
      }
      continue;
    }
    if (!big) {
      Cand e[DD_U];
#pragma unroll
      for (int u = 0; u < DD_U; ++u) {
        const uint32_t k = lo + u * DD_T + t;
        e[u] = k < hi ? ws.bcand[k] : Cand{KEY_EMPTY, 0};
      }
      for (int j = t; j < DT; j += DD_T) {
        tk[j] = 0;
        tw[j] = 0;
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < DD_U; ++u)
        if (e[u].key != KEY_EMPTY) lds_pair(tk, tw, e[u].key, e[u].w2);
      __syncthreads();
    }
    // compact the occupied slots: thread t owns slots [t Q, t Q + Q)
    constexpr int Q = DT / DD_T;
    uint32_t occ = 0;
#pragma unroll
    for (int j = 0; j < Q; ++j) occ += tk[t * Q + j] != KEY_EMPTY;
    uint32_t x = occ;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63) wt[wave] = x;
    __syncthreads();
    uint32_t pre = x - occ, total = 0;
#pragma unroll
    for (int i = 0; i < DD_T / 64; ++i) {
      pre += i < wave ? wt[i] : 0;
      total += wt[i];
    }
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const unsigned long long k = tk[t * Q + j];
      if (k != KEY_EMPTY) ws.np[lo + pre++] = NewPair{uint64_t(k), uint64_t(tw[t * Q + j])};
    }
    for (uint32_t k = lo + total + t; k < hi; k += DD_T) ws.np[k] = NewPair{KEY_EMPTY, 0};
    n_new += occ;
    __syncthreads();
  }
  ins_check_last<false>(ix, ws, 0, n_entries, n_new, 0, bad);
}

// The refreshes, when the classify pass could not do them (run by the placement's grid
// after its pairs: placement claims only empty slots, so the two never touch one value
// except an entry that both raise to the same epoch).
__device__ void refresh_pass(const DevIndex &ix, const ProbeView &pv, const InsWs &ws, uint32_t epoch) {
  const uint64_t n = pv.hdr->n;
  const uint64_t span = uint64_t(gridDim.x) * TB;
  for (uint64_t i = uint64_t(blockIdx.x) * TB + threadIdx.x; i < n; i += span) {
    const uint64_t p = ws.pos[i];
    if (!p) continue;
    uint64_t *vp = val_ptr(ix, int64_t(p - 1));
    const uint64_t v = *vp;
    if (val_epoch(v) < epoch) *vp = val_raise_epoch(v, epoch);
  }
}

// place: the distinct new pairs in bin order (so in region order), all PLACE_WG
// workgroups advancing through it together
__global__ __launch_bounds__(TB) void insp_place_kernel(DevIndex ix, ProbeView pv, InsWs ws,
                                                        const uint32_t *session, uint32_t epoch) {
  if (ws.hdr->abort) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) keep_epoch_top(ix, epoch);
  const uint64_t n = ws.hdr->n_cand;
  const uint64_t span = uint64_t(gridDim.x) * TB;
  for (uint64_t p0 = uint64_t(blockIdx.x) * TB; p0 < n; p0 += span) {  // whole workgroups iterate together
    const uint64_t p = p0 + threadIdx.x;
    int64_t tk = -1, df = -1;
    bool rf = false;
    if (p < n) {
      const NewPair e = ws.np[p];
      if (e.key != KEY_EMPTY) {
        const uint64_t w2 = np_w2(e, ws.dd);  // a fallback pair's lowest request
        bool trig;
        const int pl = place_new(ix, e.key, dd_inst(w2), epoch, session[dd_req(w2)], trig, true);
        if (pl == FAILED) set_status(ix.hdr, SMETRIC_EINTERNAL);
        else if (pl == DEFERRED) df = int64_t(p);
        else if (pl == REFRESHED) rf = true;  // a block past its probe bound that was an entry
        else if (trig) tk = int64_t(p);
      }
    }
    uncount_refreshed(ix, rf);
    append_wave(&ws.hdr->n_trig, ws.trig, ws.list_cap, tk);  // queue by np position
    append_wave(&ws.hdr->n_def, ws.def, ws.list_cap, df);
  }
  if (!ws.hdr->inl) refresh_pass(ix, pv, ws, epoch);
}

// ---------------------------------------------------------------------------------
// Insert of a small batch: one launch, one workgroup
// ---------------------------------------------------------------------------------
// A batch of a few thousand blocks is bound by launches and by one round trip to memory
// after another, not by bandwidth: the stages of the general insert (five launches)
// each find a few thousand pairs at most.  Here one workgroup takes them all, SI_U pairs
// per thread, with barriers between the stages: find every pair (from the descriptor where
// the batch was probed), dedupe the absent ones in an LDS table of pair numbers, check, then
// refresh and place.  Pairs are numbered in request order (plain) or
// carry their request (probed), so a repeated pair keeps its lowest request.  A thread
// converts the keys whose (T+1)-th plain slot it claimed and enters the pairs it had to
// defer, after a barrier each.
// One agent's requests (64 to 350 blocks each): 26 us of kernels in the eight launches that the
// self-contained insert took before, 9.3 in one.
constexpr int SI_T = 1024;
constexpr int SI_U = 4;
constexpr int SI_MAX = SI_T * SI_U;
// One launch against five (kernels alone), new pairs, in a small table and in one of 100M
// entries.  Self-contained, 64 requests of 2,048 blocks in all 26 / 31 and 52 / 45 us, of 3,072
// 35 / 28 and 70 / 46, of 4,096 48 / 35 and 95 / 56 (existing pairs 27 / 17 and 50 / 25): the line is
// at half of SI_MAX.  But its find pass takes a request by a workgroup, this kernel any pair
// by any thread: 4 requests of 3,072 blocks in all 36 / 46 and 69 / 84, of 4,096 47 / 64 and
// 91 / 112, one of 4,096 48 / 173, 16 of 4,096 48 / 33: few long requests go on to SI_MAX.  Probed
// 2,048 22 / 31 and 39 / 43, 4,096 41 / 32 and 67 / 45, and the four launches saved are 11 us of the
// host's: a replay of 64 sessions, bound by the host, 181 us with this kernel up to SI_MAX and
// 194 with half of that.
constexpr int SI_LINE = SI_MAX / 2;
constexpr int SI_LONG = 512;  // blocks per request
inline bool ins_small(int64_t n_blocks, int32_t n_req) {
  return n_req <= SI_T && n_blocks <= (n_blocks / n_req >= SI_LONG ? SI_MAX : SI_LINE);
}
constexpr int SI_TAB = 2 * SI_MAX;  // never more than half full
constexpr uint32_t SI_FREE = 0xFFFFFFFFu;

template <bool PROBED>
__global__ __launch_bounds__(SI_T) void ins_small_kernel(DevIndex ix, ProbeView pv, const uint64_t *keys,
                                                         const int64_t *blk_off, int32_t n_req, int64_t n_blocks,
                                                         const int32_t *instance, const uint32_t *session,
                                                         uint32_t epoch) {
  __shared__ uint64_t skey[SI_MAX];
  __shared__ uint32_t tab[SI_TAB];  // pair numbers
  __shared__ uint32_t sreq[SI_MAX];
  __shared__ uint16_t sinst[SI_MAX];
  __shared__ uint32_t pre[PROBED ? 1 : SI_T + 1];
  __shared__ uint32_t wt[SI_T / 64];
  __shared__ int bad_range, err;
  __shared__ unsigned int n_new, n_trig, n_def;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (t == 0) {
    bad_range = err = 0;
    n_new = n_trig = n_def = 0;
  }
  for (int h = t; h < SI_TAB; h += SI_T) tab[h] = SI_FREE;
  __syncthreads();
  uint32_t n;
  if constexpr (PROBED) {
    n = uint32_t(pv.hdr->n < uint64_t(n_blocks) ? pv.hdr->n : uint64_t(n_blocks));
    if (t == 0 && pv.hdr->err) bad_range = 1;
  } else {
    // the pairs of request r are numbered from pre[r]
    int64_t b0 = 0, nb = 0;
    if (t < n_req && !range_of(blk_off, t, n_blocks, b0, nb)) {
      bad_range = 1;
      nb = 0;
    }
    uint32_t x = uint32_t(nb);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63) wt[wave] = x;
    __syncthreads();
    uint32_t before = 0;
    n = 0;
#pragma unroll
    for (int w = 0; w < SI_T / 64; ++w) {
      before += w < wave ? wt[w] : 0;
      n += wt[w];  // at most SI_T ranges of at most SI_MAX blocks
    }
    pre[t + 1] = before + x;
    if (t == 0) {
      pre[0] = 0;
      if (n > uint64_t(n_blocks)) bad_range = 1;
    }
  }
  __syncthreads();
  if (bad_range) {
    if (t == 0) set_status(ix.hdr, SMETRIC_EINVAL);
    return;
  }
  uint64_t key[SI_U], d[SI_U];
  uint32_t r[SI_U], sess[SI_U];
  int32_t inst[SI_U];
#pragma unroll
  for (int u = 0; u < SI_U; ++u) {
    const uint32_t p = u * SI_T + t;
    key[u] = KEY_EMPTY;
    d[u] = 0;
    r[u] = 0;
    if (p < n) {
      if constexpr (PROBED) {
        key[u] = pv.part_key[p];
        r[u] = pv.part_req[p];
        d[u] = pv.desc_p[p];
      } else {
        uint32_t lo = 0, hi = uint32_t(n_req);  // pre[lo] <= p < pre[hi]
        while (hi - lo > 1) {
          const uint32_t mid = (lo + hi) >> 1;
          if (pre[mid] <= p) lo = mid;
          else hi = mid;
        }
        r[u] = lo;
        key[u] = keys[blk_off[lo] + (p - pre[lo])];
      }
    }
  }
#pragma unroll
  for (int u = 0; u < SI_U; ++u) {
    const bool in = uint32_t(u * SI_T + t) < n;
    inst[u] = in ? instance[r[u]] : 0;
    sess[u] = in ? session[r[u]] : 0;
  }
  // find: the slot of an existing pair, and whether its epoch is known to need no raise
  int64_t slot[SI_U];
  uint32_t kind[SI_U];
  bool absent[SI_U], fresh[SI_U];
#pragma unroll
  for (int u = 0; u < SI_U; ++u) {
    const uint32_t p = u * SI_T + t;
    slot[u] = -1;
    kind[u] = PLAIN;
    absent[u] = fresh[u] = false;
    if (p >= n) continue;
    skey[p] = key[u];
    sreq[p] = r[u];
    sinst[p] = uint16_t(inst[u]);
    if (inst[u] < 0 || inst[u] >= ix.n_inst || sess[u] >= SESSION_LIMIT || key[u] == KEY_EMPTY || key[u] == KEY_TOMB) {
      err = SMETRIC_EINVAL;
      continue;
    }
    const uint32_t dk = PROBED ? desc_kind(d[u]) : uint32_t(D_MANY);
    if (dk == D_ONE) {
      if (desc_inst(d[u]) == uint32_t(inst[u])) slot[u] = int64_t(desc_x(d[u]));
    } else if (dk == D_HOT || dk == D_MANY) {
      const Found f = dk == D_HOT ? find_holder(ix, desc_x(d[u]), key[u], uint32_t(inst[u]))
                                  : find_entry(ix, key[u], uint32_t(inst[u]));
      slot[u] = f.slot;
      if (f.slot >= 0) {
        kind[u] = val_kind(f.val);
        fresh[u] = val_epoch(f.val) >= epoch;
      }
    }
    absent[u] = slot[u] < 0;
  }
  __syncthreads();
  if (err) {
    if (t == 0) set_status(ix.hdr, err);
    return;
  }
  // dedupe: a slot of the table ends with the number of its pair that has the lowest request
  uint32_t own[SI_U];
#pragma unroll
  for (int u = 0; u < SI_U; ++u) {
    const uint32_t p = u * SI_T + t;
    own[u] = 0;
    if (!absent[u]) continue;
    uint32_t h = uint32_t(mix64(key[u] ^ ((uint64_t(inst[u]) + 1) * 0xC2B2AE3D27D4EB4Full))) & (SI_TAB - 1);
    while (true) {
      uint32_t cur = atomicCAS(&tab[h], SI_FREE, p);
      if (cur == SI_FREE) break;
      if (skey[cur] == key[u] && sinst[cur] == uint16_t(inst[u])) {
        // the same pair (whichever of its numbers the slot holds by now): the lower request stays
        while (sreq[cur] > r[u] || (sreq[cur] == r[u] && cur > p)) {
          const uint32_t was = atomicCAS(&tab[h], cur, p);
          if (was == cur) break;
          cur = was;
        }
        break;
      }
      h = (h + 1) & (SI_TAB - 1);
    }
    own[u] = h;
  }
  __syncthreads();
  uint32_t mine = 0;
#pragma unroll
  for (int u = 0; u < SI_U; ++u) {
    absent[u] = absent[u] && tab[own[u]] == uint32_t(u * SI_T + t);
    mine += absent[u];
  }
  if (mine) atomicAdd(&n_new, mine);
  __syncthreads();
  if (t == 0) {
    if (ix.hdr->n_entries + n_new > ix.capacity) {
      err = SMETRIC_EFULL;
      set_status(ix.hdr, SMETRIC_EFULL);
    } else if (n_new) {
      atomicAdd(&ix.hdr->n_entries, (unsigned long long)n_new);
    }
  }
  __syncthreads();
  if (err) return;
  if (t == 0) keep_epoch_top(ix, epoch);
  uint32_t trig = 0, def = 0;  // bit u: pair u converts its key, was deferred
#pragma unroll
  for (int u = 0; u < SI_U; ++u) {
    bool rf = false;
    if (slot[u] >= 0) {
      if (!fresh[u]) raise_epoch_at(val_ptr(ix, slot[u]), kind[u], uint32_t(inst[u]), epoch);
    } else if (absent[u]) {
      bool tr;
      const int pl = place_new(ix, key[u], uint32_t(inst[u]), epoch, sess[u], tr, true);
      if (pl == FAILED) set_status(ix.hdr, SMETRIC_EINTERNAL);
      else if (pl == DEFERRED) def |= 1u << u;
      else if (pl == REFRESHED) rf = true;  // a block past its probe bound that was an entry
      else if (tr) trig |= 1u << u;
    }
    uncount_refreshed(ix, rf);
  }
  if (trig) n_trig = 1;
  if (def) n_def = 1;
  __syncthreads();
  if (n_trig) {  // every claim and value above is visible before a conversion reads the chain
    __threadfence();
    while (trig) {
      const int u = __builtin_ctz(trig);
      trig &= trig - 1;
      if (!spill_key(ix, skey[u * SI_T + t])) set_status(ix.hdr, SMETRIC_EINTERNAL);
    }
    __threadfence();
    __syncthreads();
  }
  if (n_def) {
    __threadfence();
    while (__ballot(def != 0)) {
      bool rf = false;
      if (def) {
        const int u = __builtin_ctz(def);
        def &= def - 1;
        const uint32_t p = u * SI_T + t;
        bool tr;
        const int pl = place_new(ix, skey[p], sinst[p], epoch, session[sreq[p]], tr, false);
        rf = pl == REFRESHED;
        if (pl != PLACED && pl != REFRESHED) set_status(ix.hdr, SMETRIC_EINTERNAL);
      }
      uncount_refreshed(ix, rf);
    }
  }
}

// ---------------------------------------------------------------------------------
// Evict / dump
// ---------------------------------------------------------------------------------
// A tile of the table, TILE buckets: lane l of a wavefront takes slot l of its 8 buckets, so
// that a load instruction covers eight 64-byte runs; a thread of NT holds TILE * SLOTS / NT
// slots, their loads issued together, from one scalar base (an address each would take as
// many registers as the data).
constexpr int TILE = 512;
template <int NT>
__device__ __forceinline__ uint32_t tile_word(int u) {  // its key's word in the tile
  const uint32_t i = uint32_t(u * NT) + threadIdx.x;
  return (i / SLOTS) * BUCKET_WORDS + i % SLOTS;
}
__device__ __forceinline__ uint32_t tile_words(const DevIndex &ix, uint64_t b0) {
  return uint32_t(ix.n_buckets - b0 < TILE ? ix.n_buckets - b0 : TILE) * BUCKET_WORDS;
}
template <int NT>
__device__ __forceinline__ void load_tile(const DevIndex &ix, uint64_t b0, uint64_t *k, uint64_t *v) {
  const uint64_t *base = ix.slots + b0 * BUCKET_WORDS;
  const uint32_t nw = tile_words(ix, b0);
#pragma unroll
  for (int u = 0; u < TILE * SLOTS / NT; ++u) {
    const uint32_t w = tile_word<NT>(u), at = w < nw ? w : 0;
    k[u] = base[at];
    v[u] = base[at + SLOTS];
    if (w >= nw) k[u] = KEY_EMPTY;
  }
}
__device__ __forceinline__ bool is_entry(uint64_t k, uint64_t v) {  // a plain or member slot
  return k != KEY_EMPTY && k != KEY_TOMB && val_kind(v) != HEADER;
}

// All live entries for the dump, which sorts them: a workgroup reserves its tile's output
// with one atomic (one per entry made a single counter the bottleneck).
__global__ __launch_bounds__(TB) void gather_kernel(DevIndex ix, uint64_t *keys, uint64_t *vals,
                                                    unsigned long long *count, uint64_t cap) {
  constexpr int GS = TILE * SLOTS / TB;
  static_assert(GS * (TB / 64) == 64, "a round's ballots: one per lane of the scan");
  __shared__ uint32_t pre[64];
  __shared__ unsigned long long wg_base;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint64_t b0 = uint64_t(blockIdx.x) * TILE; b0 < ix.n_buckets; b0 += uint64_t(gridDim.x) * TILE) {
    uint64_t k[GS], v[GS], live[GS];
    load_tile<TB>(ix, b0, k, v);
#pragma unroll
    for (int u = 0; u < GS; ++u) {
      live[u] = __ballot(is_entry(k[u], v[u]));
      if (lane == 0) pre[u * (TB / 64) + wave] = uint32_t(__popcll(live[u]));
    }
    __syncthreads();
    if (wave == 0) {  // exclusive prefix of the ballots' counts
      const uint32_t c = pre[lane];
      uint32_t x = c;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
      }
      pre[lane] = x - c;
      if (lane == 63) wg_base = x ? atomicAdd(count, (unsigned long long)x) : 0;
    }
    __syncthreads();
    const unsigned long long base = wg_base;
#pragma unroll
    for (int u = 0; u < GS; ++u) {
      const unsigned long long at = base + pre[u * (TB / 64) + wave] + __popcll(live[u] & ((uint64_t(1) << lane) - 1));
      if (((live[u] >> lane) & 1) && at < cap) {
        keys[at] = k[u];
        vals[at] = val_dump(v[u]);
      }
    }
    __syncthreads();  // pre and wg_base are reused
  }
}

// The header slot of a key with a bitmap record (-1: none); it lies in the key's chain.
__device__ int64_t find_header(const DevIndex &ix, uint64_t key) {
  uint64_t b = home_bucket(key, ix.n_buckets);
  for (uint64_t step = 0; step < ix.n_buckets; ++step, b = next_bucket(b, ix.n_buckets)) {
    const uint64_t *bk = ix.slots + b * BUCKET_WORDS;
    for (int s = 0; s < SLOTS; ++s) {
      const uint64_t k = bk[s];
      if (k == KEY_EMPTY) return -1;
      if (k == key && val_kind(bk[SLOTS + s]) == HEADER) return int64_t(b * SLOTS + s);
    }
  }
  return -1;
}

// Eviction as a selection: the cut is the m-th smallest entry under (epoch, key, instance),
// and every entry up to it leaves.  That order as two words, of a key and a value in the
// dump's format (instance << 48 | epoch << 24 | session):
struct SelCut {
  uint64_t hi, lo;
};
__host__ __device__ __forceinline__ uint64_t sel_hi(uint64_t key, uint32_t epoch) {
  return (uint64_t(epoch) << 40) | (key >> 24);
}
__device__ __forceinline__ bool sel_leaves(uint64_t key, uint64_t hi, uint32_t inst, const SelCut &c) {
  return hi < c.hi || (hi == c.hi && (((key & 0xFFFFFF) << 16) | inst) <= c.lo);
}
// The entries near the cut are settled digit by digit -- epoch in two 11-bit digits, the key
// in five 12-bit digits and a last 4-bit part joined with the instance's top 6 bits, then the
// instance's low 10 bits -- each digit fixed by one histogram pass over the entries that
// share the digits fixed so far, until the whole of a bin goes.
constexpr int SEL_LEVELS = 9;
constexpr int SEL_BINS = 4096;
struct SelPrefix {
  int level;  // digits fixed so far
  uint32_t digit[SEL_LEVELS];
};
__host__ __device__ __forceinline__ uint32_t sel_digit(uint64_t key, uint64_t v, int l) {
  const uint32_t ep = dump_epoch(v), inst = dump_inst(v);
  switch (l) {
    case 0: return ep >> 11;
    case 1: return ep & 0x7FFu;
    case 2: return uint32_t(key >> 52);
    case 3: return uint32_t(key >> 40) & 0xFFFu;
    case 4: return uint32_t(key >> 28) & 0xFFFu;
    case 5: return uint32_t(key >> 16) & 0xFFFu;
    case 6: return uint32_t(key >> 4) & 0xFFFu;
    case 7: return (uint32_t(key & 15) << 6) | (inst >> 10);
    default: return inst & 0x3FFu;
  }
}
__device__ __forceinline__ bool sel_on(uint64_t key, uint64_t v, const SelPrefix &p) {
  for (int l = 0; l < p.level; ++l)
    if (sel_digit(key, v, l) != p.digit[l]) return false;
  return true;
}
// The largest (epoch, key, instance) on the prefix, but not past `hi`, the end of the range
// that the entries were taken from: the prefix may reach beyond it.
__host__ __device__ inline SelCut sel_cut(const SelPrefix &p, uint64_t hi) {
  uint64_t d[SEL_LEVELS];
  for (int l = 0; l < SEL_LEVELS; ++l) d[l] = l < p.level ? p.digit[l] : l == 1 ? 0x7FF : l >= 7 ? 0x3FF : 0xFFF;
  const uint64_t key =
      (d[2] << 52) | (d[3] << 40) | (d[4] << 28) | (d[5] << 16) | (d[6] << 4) | (d[7] >> 6);
  const SelCut c = {sel_hi(key, uint32_t((d[0] << 11) | d[1])),
                    ((key & 0xFFFFFF) << 16) | ((d[7] & 63) << 10) | d[8]};
  return c.hi > hi ? SelCut{hi, ~uint64_t(0)} : c;
}

// The eviction's counters, in its workspace.
struct EvictState {
  unsigned long long n_entries;               // as the header has it
  unsigned long long lo, hi;                  // the range of sel_hi that the scan copies out
  unsigned long long n_in, n_fin;             // copied by the scan; of these, for the last passes
  unsigned long long n_left, n_trig, n_def;   // the rebuild's lists
  SelCut cut;                                 // once a kernel decides it
};
// The scan's counters: entries, tombstones, entries below the range.  One atomic takes 12 ns
// on one address, so the workgroups spread over EV_LANES lines, which the host adds up.
constexpr int EV_LANES = 8, EV_LINE = 16;

// Entries of a wavefront collected in LDS and written out some hundreds at a time, each
// batch with one reservation.
constexpr int STAGE = 512;
struct WaveStage {
  uint64_t k[TB / 64][STAGE], v[TB / 64][STAGE];
  uint32_t n[TB / 64];
  unsigned long long base;
};
__device__ __forceinline__ void stage_push(WaveStage &st, uint32_t &n, bool mine, uint64_t k, uint64_t v,
                                           unsigned long long *count, uint64_t *ck, uint64_t *cv, uint64_t cap) {
  const uint64_t b = __ballot(mine);
  if (!b) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t c = uint32_t(__popcll(b));
  if (n + c > STAGE) {
    unsigned long long at = 0;
    if (lane == 0) at = atomicAdd(count, (unsigned long long)n);
    at = __shfl(at, 0, 64);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (uint32_t i = lane; i < n; i += 64)
      if (at + i < cap) {
        ck[at + i] = st.k[wave][i];
        cv[at + i] = st.v[wave][i];
      }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    n = 0;
  }
  if (mine) {
    const uint32_t at = n + uint32_t(__popcll(b & ((uint64_t(1) << lane) - 1)));
    st.k[wave][at] = k;
    st.v[wave][at] = v;
  }
  n += c;
}
__device__ __forceinline__ void stage_flush(WaveStage &st, uint32_t n, unsigned long long *count, uint64_t *ck,
                                            uint64_t *cv, uint64_t cap) {  // the whole workgroup
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) st.n[wave] = n;
  __syncthreads();
  uint32_t before = 0, total = 0;
  for (int w = 0; w < TB / 64; ++w) {
    if (w < wave) before += st.n[w];
    total += st.n[w];
  }
  if (threadIdx.x == 0) st.base = total ? atomicAdd(count, (unsigned long long)total) : 0;
  __syncthreads();
  const uint64_t at = st.base + before;
  for (uint32_t i = lane; i < n; i += 64)
    if (at + i < cap) {
      ck[at + i] = st.k[wave][i];
      cv[at + i] = st.v[wave][i];
    }
}

// The bin of the 4,096 in h that holds the left-th smallest (1-based), by a whole workgroup
// of FIN_T: its index (SEL_BINS: none), the count below it and its own.
constexpr int FIN_T = 1024;
struct BinPick {
  uint32_t wt[FIN_T / 64];
  uint32_t bin, below, count;
};
__device__ __forceinline__ void pick_bin(const uint32_t *h, uint32_t left, BinPick &s) {
  constexpr int PER = SEL_BINS / FIN_T;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  uint32_t c[PER], sum = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    c[j] = h[t * PER + j];
    sum += c[j];
  }
  uint32_t x = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) s.wt[wave] = x;
  if (t == 0) s.bin = SEL_BINS;
  __syncthreads();
  uint32_t below = x - sum;
  for (int w = 0; w < wave; ++w) below += s.wt[w];
  if (below < left && left <= below + sum) {  // one thread
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (below < left && left <= below + c[j]) {
        s.bin = uint32_t(t * PER + j);
        s.below = below;
        s.count = c[j];
      }
      below += c[j];
    }
  }
  __syncthreads();
}

// Where the cut lies, roughly, from a sample: EV_SAMPLE buckets evenly over the table (keys
// are hashes, but a key's home bucket follows its top bits).  It also clears the counters.
// Without a sample the range is everything.  In an empty index this pass and the two after it
// stop at the header's count (2^28 slots: 770 us -> 31; a header read by the host alone is 26,
// but would come before every other eviction).
constexpr int EV_SAMPLE = 4096;
__global__ __launch_bounds__(TB) void evict_sample_kernel(DevIndex ix, EvictState *st, unsigned long long *counts,
                                                          uint64_t *sample) {
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      EvictState z{};
      z.n_entries = ix.hdr->n_entries;
      z.hi = ~0ull;
      *st = z;
    }
    if (threadIdx.x < EV_LANES * EV_LINE) counts[threadIdx.x] = 0;
  }
  if (!sample || ix.hdr->n_entries == 0) return;
  const uint32_t i = blockIdx.x * TB + threadIdx.x;  // EV_SAMPLE * SLOTS threads
  const uint64_t b = (uint64_t(i / SLOTS) * ix.n_buckets) / EV_SAMPLE;
  const uint64_t *p = ix.slots + b * BUCKET_WORDS + i % SLOTS;
  const uint64_t k = p[0], v = p[SLOTS];
  sample[i] = is_entry(k, v) ? sel_hi(k, val_epoch(v)) : ~uint64_t(0);
}
// The range for the scan: from the bin of the sample's order statistic six standard
// deviations below the cut's expected rank to the bin of the one as far above it (and 16 on
// each side, for entries of one key that lie together).  A range that misses the cut shows
// in the scan's counts.  One workgroup, the sample in registers, radix digits in LDS.
__global__ __launch_bounds__(FIN_T) void evict_range_kernel(const uint64_t *__restrict__ sample, uint32_t frac_num,
                                                            uint32_t frac_den, EvictState *st) {
  constexpr int PER = EV_SAMPLE * SLOTS / FIN_T;
  __shared__ uint32_t h[SEL_BINS];
  __shared__ BinPick bp;
  __shared__ unsigned long long s_or, s_and;
  __shared__ uint32_t s_n;
  if (st->n_entries == 0) return;
  const int t = threadIdx.x;
  uint64_t x[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) x[u] = sample[u * FIN_T + t];
  if (t == 0) {
    s_or = s_n = 0;
    s_and = ~0ull;
  }
  __syncthreads();
  uint64_t o = 0, a = ~uint64_t(0);
  uint32_t c = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (x[u] != ~uint64_t(0)) {
      o |= x[u];
      a &= x[u];
      ++c;
    }
  atomicOr(&s_or, (unsigned long long)o);
  atomicAnd(&s_and, (unsigned long long)a);
  atomicAdd(&s_n, c);
  __syncthreads();
  const uint32_t n = s_n;
  if (n == 0) return;  // the range stays everything
  const uint64_t diff = s_or ^ s_and;
  const double q = double(frac_num) / double(frac_den), r = q * double(n);
  const double dev = 6.0 * sqrt(double(n) * q * (1.0 - q)) + 16.0;
  for (int side = 0; side < 2; ++side) {
    const double rr = side ? r + dev + 1.0 : r - dev;
    if (rr < 1.0 || rr > double(n)) continue;  // open on this side
    uint32_t left = uint32_t(rr);
    int shift = diff ? 64 - __clzll((long long)diff) : 0;  // bits below are not fixed yet (at most 62)
    uint64_t pre = s_or >> shift;
    uint32_t on = n;
    while (shift > 0 && on > 8) {
      const int w = shift < 12 ? shift : 12;
      for (int b = t; b < SEL_BINS; b += FIN_T) h[b] = 0;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < PER; ++u)
        if (x[u] != ~uint64_t(0) && (x[u] >> shift) == pre)
          atomicAdd(&h[uint32_t(x[u] >> (shift - w)) & ((1u << w) - 1u)], 1u);
      __syncthreads();
      pick_bin(h, left, bp);
      left -= bp.below;
      on = bp.count;
      shift -= w;
      pre = (pre << w) | bp.bin;
      __syncthreads();
    }
    if (t == 0) {
      if (side) st->hi = ((pre + 1) << shift) - 1;
      else st->lo = pre << shift;
    }
  }
}

// The one pass that decides: the whole table read once, its entries and tombstones counted,
// those below the range counted and those in it copied out.  Bound by the read of 128 bytes
// a bucket: 50M entries in 9.5M buckets 238 us, 5.1 TB/s.  (Gathering every entry with its
// slot and selecting over the gathered arrays moved those bytes four times: 851 us and two
// passes of 229 to 468 us.)
__global__ __launch_bounds__(TB) void evict_scan_kernel(DevIndex ix, EvictState *st, unsigned long long *counts,
                                                        uint64_t *ck, uint64_t *cv, uint64_t cap) {
  __shared__ WaveStage stage;
  __shared__ uint32_t wc[TB / 64][3];
  if (st->n_entries == 0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lo = st->lo, hi = st->hi;
  constexpr int GS = TILE * SLOTS / TB;
  uint32_t live = 0, tombs = 0, below = 0, staged = 0;
  for (uint64_t b0 = uint64_t(blockIdx.x) * TILE; b0 < ix.n_buckets; b0 += uint64_t(gridDim.x) * TILE) {
    uint64_t k[GS], v[GS];
    load_tile<TB>(ix, b0, k, v);
#pragma unroll
    for (int u = 0; u < GS; ++u) {
      const bool e = is_entry(k[u], v[u]);
      const uint64_t a = sel_hi(k[u], val_epoch(v[u]));
      live += e;
      tombs += k[u] == KEY_TOMB;
      below += e && a < lo;
      stage_push(stage, staged, e && a >= lo && a <= hi, k[u], val_dump(v[u]), &st->n_in, ck, cv, cap);
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    live += __shfl_xor(live, d, 64);
    tombs += __shfl_xor(tombs, d, 64);
    below += __shfl_xor(below, d, 64);
  }
  if (lane == 0) {
    wc[wave][0] = live;
    wc[wave][1] = tombs;
    wc[wave][2] = below;
  }
  stage_flush(stage, staged, &st->n_in, ck, cv, cap);
  if (threadIdx.x < 3) {
    unsigned long long x = 0;
    for (int w = 0; w < TB / 64; ++w) x += wc[w][threadIdx.x];
    if (x) atomicAdd(&counts[(blockIdx.x % EV_LANES) * EV_LINE + threadIdx.x], x);
  }
}

// One selection pass: the histogram of the next digit over the entries on the prefix.
__global__ __launch_bounds__(TB) void sel_hist_kernel(const uint64_t *__restrict__ keys,
                                                      const uint64_t *__restrict__ vals, uint64_t n, SelPrefix p,
                                                      unsigned long long *hist) {
  __shared__ uint32_t h[SEL_BINS];
  for (int b = threadIdx.x; b < SEL_BINS; b += TB) h[b] = 0;
  __syncthreads();
  const uint64_t stride = uint64_t(gridDim.x) * TB;
  for (uint64_t i = uint64_t(blockIdx.x) * TB + threadIdx.x; i < n; i += stride) {
    const uint64_t k = keys[i], v = vals[i];
    if (sel_on(k, v, p)) atomicAdd(&h[sel_digit(k, v, p.level)], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < SEL_BINS; b += TB)
    if (h[b]) atomicAdd(&hist[b], (unsigned long long)h[b]);
}

// The entries on the prefix, few enough for one workgroup, copied out for it.
__global__ __launch_bounds__(TB) void sel_copy_kernel(const uint64_t *__restrict__ keys,
                                                      const uint64_t *__restrict__ vals, uint64_t n, SelPrefix p,
                                                      unsigned long long *count, uint64_t *ck, uint64_t *cv,
                                                      uint64_t cap) {
  __shared__ WaveStage stage;
  uint32_t staged = 0;
  const uint64_t stride = uint64_t(gridDim.x) * TB;
  for (uint64_t i0 = uint64_t(blockIdx.x) * TB; i0 < n; i0 += stride) {  // whole wavefronts iterate together
    const uint64_t i = i0 + threadIdx.x;
    const uint64_t k = keys[i < n ? i : 0], v = vals[i < n ? i : 0];
    stage_push(stage, staged, i < n && sel_on(k, v, p), k, v, count, ck, cv, cap);
  }
  stage_flush(stage, staged, count, ck, cv, cap);
}

// The selection's last passes over at most SEL_FIN entries, by one workgroup and without the
// host (a pass with the host in it costs 25 us): each remaining digit's histogram in LDS and
// its bin, until the whole bin goes; the cut is left in st.  Passes read the entries in
// rounds of FIN_U per thread, loads issued together; once FIN_L or fewer are on the prefix
// they are kept in LDS.  n_c, when given, is the number that was copied out: it has to be n.
constexpr uint64_t SEL_FIN = uint64_t(1) << 16;
constexpr int FIN_U = 8, FIN_L = 1024;
__global__ __launch_bounds__(FIN_T) void sel_finish_kernel(DevIndex ix, const uint64_t *__restrict__ keys,
                                                           const uint64_t *__restrict__ vals, uint64_t n, SelPrefix p,
                                                           unsigned long long rem, unsigned long long on_prefix,
                                                           const unsigned long long *n_c, EvictState *st) {
  __shared__ SelPrefix sp;
  __shared__ uint32_t h[SEL_BINS];
  __shared__ uint64_t lk[FIN_L], lv[FIN_L];
  __shared__ BinPick bp;
  __shared__ uint32_t n_list;
  static_assert(FIN_L <= FIN_T, "one listed entry per thread");
  const int t = threadIdx.x;
  if (t == 0) {
    sp = p;
    n_list = 0;
  }
  const bool whole = !n_c || *n_c == n;
  int level = p.level;
  uint32_t left = uint32_t(rem), on = uint32_t(on_prefix);  // at most SEL_FIN
  bool listed = false;
  while (whole && level < SEL_LEVELS && left < on) {
    for (int b = t; b < SEL_BINS; b += FIN_T) h[b] = 0;
    __syncthreads();
    if (listed) {
      if (uint32_t(t) < n_list && sel_on(lk[t], lv[t], sp)) atomicAdd(&h[sel_digit(lk[t], lv[t], level)], 1u);
    } else {
      for (uint64_t i0 = 0; i0 < n; i0 += FIN_T * FIN_U) {
        uint64_t k[FIN_U], v[FIN_U];
#pragma unroll
        for (int u = 0; u < FIN_U; ++u) {
          const uint64_t i = i0 + u * FIN_T + t;
          k[u] = keys[i < n ? i : 0];
          v[u] = vals[i < n ? i : 0];
        }
#pragma unroll
        for (int u = 0; u < FIN_U; ++u) {
          if (i0 + u * FIN_T + t >= n || !sel_on(k[u], v[u], sp)) continue;
          atomicAdd(&h[sel_digit(k[u], v[u], level)], 1u);
          if (on <= FIN_L) {
            const uint32_t at = atomicAdd(&n_list, 1u);
            if (at < FIN_L) {
              lk[at] = k[u];
              lv[at] = v[u];
            }
          }
        }
      }
      listed = on <= FIN_L;
    }
    __syncthreads();
    pick_bin(h, left, bp);
    if (bp.bin == SEL_BINS) break;  // fewer entries on the prefix than counted before
    left -= bp.below;
    on = bp.count;
    ++level;
    if (t == 0) {
      sp.digit[level - 1] = bp.bin;
      sp.level = level;
    }
    __syncthreads();
  }
  if (t == 0) {
    if (!whole || left != on) set_status(ix.hdr, SMETRIC_EINTERNAL);  // the full tuple is unique
    st->cut = sel_cut(sp, st->hi);
  }
}

// Rebuild, second pass: the entries the tile pass left, one per thread (all survivors).
// Claims that trigger a key's conversion or are deferred are queued by their place in the
// list for the spill and deferred passes; nearly all members are deferred, so a workgroup
// queues its own with one atomic.  The list is in the order of the tiles, more or less, so few
// workgroups keep the part of the table that is walked at one time small: a third of 76M
// entries, 16M of them members, 5.7 ms with 4,096 workgroups (and an atomic per wavefront), 1.8
// with 512, 1.6 with 384, 2.0 with 256; of 155M, 5M of them members, 2.2, 1.4, 0.9 and 1.1.  (From
// lists per tile, a workgroup each, 4.8 and 1.9.)
constexpr int CLAIM_WG = 384;
__global__ __launch_bounds__(TB) void rebuild_claim_kernel(DevIndex ix, const uint64_t *__restrict__ keys,
                                                           const uint64_t *__restrict__ vals,
                                                           const unsigned long long *n_left, uint64_t *trig,
                                                           unsigned long long *n_trig, uint64_t *def,
                                                           unsigned long long *n_def, uint64_t cap) {
  __shared__ uint32_t wc[TB / 64];
  __shared__ unsigned long long base;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t n = *n_left < cap ? *n_left : cap;
  for (uint64_t i0 = uint64_t(blockIdx.x) * TB; i0 < n; i0 += uint64_t(gridDim.x) * TB) {
    const uint64_t i = i0 + threadIdx.x;
    int64_t tk = -1, df = -1;
    if (i < n) {
      const uint64_t k = keys[i], v = vals[i];
      bool trg;
      const int pl = place_new(ix, k, dump_inst(v), dump_epoch(v), dump_session(v), trg, true);
      if (pl == FAILED || pl == REFRESHED) set_status(ix.hdr, SMETRIC_EINTERNAL);  // survivors are distinct
      else if (pl == DEFERRED) df = int64_t(i);
      else if (trg) tk = int64_t(i);
    }
    append_wave(n_trig, trig, cap, tk);
    const uint64_t want = __ballot(df >= 0);
    if (lane == 0) wc[wave] = uint32_t(__popcll(want));
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < TB / 64; ++w) {
      before += w < wave ? wc[w] : 0u;
      total += wc[w];
    }
    if (threadIdx.x == 0 && total) base = atomicAdd(n_def, (unsigned long long)total);
    __syncthreads();
    const unsigned long long at = base + before + __popcll(want & ((uint64_t(1) << lane) - 1));
    if (df >= 0 && at < cap) def[at] = uint64_t(df);
  }
}

// Rebuild, first pass: workgroup k rewrites the whole of the table's tile k in place,
// assembled in LDS: the entries above the cut whose home bucket lies in the tile are placed
// without a walk.  With c(b) of them homed at bucket b, home b's entries
// take the consecutive slots from S(b) on, S(b) = max(SLOTS b, S(b - 1) + c(b - 1)), i.e.
// with P the exclusive prefix sum of c, S(b) = P(b) + max over j <= b of (SLOTS j - P(j)).
// Every slot from an entry's home bucket up to its own is then taken, as linear probing
// requires, and the class bit of each entry past its home bucket goes into that bucket's
// mask.  Everything else -- members (a key's plain slots are capped at T + 1 before its
// conversion, which the claim pass enforces), entries homed in another tile, entries past
// the tile's last slot -- is copied to the list that the claim pass enters from the home
// buckets of the written table.  Bound by the table's read and write, 128 bytes a bucket
// each way, two workgroups' tiles to a compute unit's LDS: a third of 47.5M entries 473 us,
// 5.1 TB/s (560 us from gathered entries; a workgroup of 256 takes so many registers for its
// 16 slots a thread that one runs on a compute unit: 1,040 us).
__global__ __launch_bounds__(TILE) void rebuild_tile_kernel(DevIndex ix, SelCut cut_host, const SelCut *cut_dev,
                                                          uint64_t *lk, uint64_t *lv, unsigned long long *n_left,
                                                          uint64_t cap, unsigned long long n_entries) {
  const SelCut cut = cut_dev ? *cut_dev : cut_host;
  constexpr int RT = TILE, GS = SLOTS;  // one bucket per thread in the scans, SLOTS slots to place
  constexpr uint32_t GONE = RT, LEFT = RT + 1;
  __shared__ uint64_t tb[RT * BUCKET_WORDS];  // the tile: keys, then values, per bucket
  __shared__ uint32_t tm[RT];                 // the tile's displacement masks
  __shared__ uint32_t hc[RT];                 // entries homed at each bucket, then S(b)
  __shared__ uint32_t wsum[RT / 64], wmax[RT / 64];
  __shared__ uint32_t n_lo;
  __shared__ unsigned long long lo_base;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint64_t b_lo = uint64_t(blockIdx.x) * RT;
  const uint64_t nb = ix.n_buckets - b_lo < uint64_t(RT) ? ix.n_buckets - b_lo : uint64_t(RT);
  if (blockIdx.x == 0 && t == 0) {
    ix.hdr->n_entries = n_entries;
    ix.hdr->rec_used = 0;
  }
  uint64_t k[GS], v[GS];
  load_tile<RT>(ix, b_lo, k, v);
  for (int i = t; i < RT * BUCKET_WORDS; i += RT) tb[i] = (i % BUCKET_WORDS) < SLOTS ? KEY_EMPTY : VAL_UNSET;
  for (int i = t; i < RT; i += RT) tm[i] = hc[i] = 0;
  if (t == 0) n_lo = 0;
  __syncthreads();
  // survivors homed in the tile count themselves at their home (the count is their rank
  // there), the rest are listed
  uint32_t home[GS], rank[GS];  // home: offset in the tile, or GONE or LEFT (rank: place in the list)
#pragma unroll
  for (int u = 0; u < GS; ++u) {
    home[u] = GONE;
    rank[u] = 0;
    if (is_entry(k[u], v[u]) && !sel_leaves(k[u], sel_hi(k[u], val_epoch(v[u])), val_inst(v[u]), cut)) {
      const uint64_t h = home_bucket(k[u], ix.n_buckets);
      if (val_kind(v[u]) != MEMBER && h >= b_lo && h < b_lo + nb) {
        home[u] = uint32_t(h - b_lo);
        rank[u] = atomicAdd(&hc[home[u]], 1u);
      } else {
        home[u] = LEFT;
        rank[u] = atomicAdd(&n_lo, 1u);
      }
    }
  }
  __syncthreads();
  // S(b) over the tile, thread t holding bucket t: exclusive sums P and running maxima of
  // SLOTS j - P(j) across the workgroup (wavefront scans, then the waves' totals)
  const uint32_t c = hc[t];
  uint32_t sum = c;  // inclusive prefix sum over the threads
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(sum, d, 64);
    if (lane >= d) sum += y;
  }
  if (lane == 63) wsum[wave] = sum;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave; ++w) before += wsum[w];
  const uint32_t pt = before + sum - c;  // P(t)
  int32_t m = int32_t(SLOTS * t) - int32_t(pt);
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int32_t y = __shfl_up(m, d, 64);
    if (lane >= d && y > m) m = y;
  }
  if (lane == 63) wmax[wave] = uint32_t(m);
  __syncthreads();
  for (int w = 0; w < wave; ++w) m = int32_t(wmax[w]) > m ? int32_t(wmax[w]) : m;
  hc[t] = uint32_t(int32_t(pt) + m);  // S(t): only thread t reads c(t)
  __syncthreads();
#pragma unroll
  for (int u = 0; u < GS; ++u) {
    if (home[u] >= RT) continue;
    const uint32_t at = hc[home[u]] + rank[u];  // slot index in the tile
    if (at >= uint32_t(nb) * SLOTS) {           // past the tile's last slot
      rank[u] = atomicAdd(&n_lo, 1u);
      home[u] = LEFT;
      continue;
    }
    const uint32_t b = at / SLOTS, s = at % SLOTS;
    tb[b * BUCKET_WORDS + s] = k[u];
    tb[b * BUCKET_WORDS + SLOTS + s] = make_val(val_inst(v[u]), PLAIN, val_epoch(v[u]), val_session(v[u]));
    if (b > home[u]) atomicOr(&tm[home[u]], 1u << (2 * key_cls(k[u]) + (b == home[u] + 1 ? 0 : 1)));
  }
  __syncthreads();
  if (t == 0) lo_base = n_lo ? atomicAdd(n_left, (unsigned long long)n_lo) : 0;
  for (uint64_t i = t; i < nb; i += RT) {
    if (MASK_W == 16) reinterpret_cast<uint16_t *>(ix.mask)[b_lo + i] = uint16_t(tm[i]);
    else ix.mask[b_lo + i] = uint8_t(tm[i]);
  }
  ulonglong2 *dst = reinterpret_cast<ulonglong2 *>(ix.slots + b_lo * BUCKET_WORDS);
  const ulonglong2 *src = reinterpret_cast<const ulonglong2 *>(tb);
  for (uint64_t w = t; w < nb * (BUCKET_WORDS / 2); w += RT) dst[w] = src[w];
  __syncthreads();
  const uint64_t base = lo_base;
#pragma unroll
  for (int u = 0; u < GS; ++u)
    if (home[u] == LEFT && base + rank[u] < cap) {
      lk[base + rank[u]] = k[u];
      lv[base + rank[u]] = val_dump(v[u]);
    }
}

// Enter the deferred pairs once their keys are converted (or, with the pool exhausted,
// as further plain slots).  Items index `keys` (and `vals`) directly, or through
// `via` into the dedupe table `dd` (insert: session of the lowest request).
__global__ void deferred_kernel(DevIndex ix, const uint64_t *items, const unsigned long long *n_items,
                                const int *abort_flag, const DSlot *dd, const uint32_t *session, uint32_t epoch,
                                const uint64_t *keys, const uint64_t *vals, const NewPair *np) {
  if (abort_flag && *abort_flag) return;
  const uint64_t n = *n_items;
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
    const uint64_t t = items[i];
    bool trig;
    int pl;
    if (np) {
      const NewPair e = np[t];
      const uint64_t w2 = np_w2(e, dd);
      pl = place_new(ix, e.key, dd_inst(w2), epoch, session[dd_req(w2)], trig, false);
    } else if (dd) {
      const DSlot d = dd[t];
      pl = place_new(ix, d.key, dd_inst(d.w2), epoch, session[dd_req(d.w2)], trig, false);
    } else {
      const uint64_t v = vals[t];
      pl = place_new(ix, keys[t], dump_inst(v), dump_epoch(v), dump_session(v), trig, false);
    }
    if (pl == REFRESHED && !np && !dd) pl = FAILED;  // rebuild survivors are distinct
    if (pl != PLACED && pl != REFRESHED) set_status(ix.hdr, SMETRIC_EINTERNAL);
    uncount_refreshed(ix, pl == REFRESHED);
  }
}

// Eviction in place: the entries at or below the cut become tombstones (a member also
// leaves its key's bitmap); every other entry keeps its slot.  Tombstones are never
// reclaimed by inserts, so the caller rebuilds the table instead once they would pass an
// eighth of the slots.  Values first, and the keys of those alone whose epoch the cut
// reaches: where few leave, most of the keys' halves of the buckets are not read (5 % of 50M
// entries: 288 us; 322 us with twice the slots a thread).
constexpr int TT = 512;
__global__ __launch_bounds__(TT) void evict_tomb_kernel(DevIndex ix, SelCut cut_host, const SelCut *cut_dev,
                                                        unsigned long long n_left) {
  const SelCut cut = cut_dev ? *cut_dev : cut_host;
  constexpr int GS = TILE * SLOTS / TT;
  if (blockIdx.x == 0 && threadIdx.x == 0) ix.hdr->n_entries = n_left;
  for (uint64_t b0 = uint64_t(blockIdx.x) * TILE; b0 < ix.n_buckets; b0 += uint64_t(gridDim.x) * TILE) {
    uint64_t *base = ix.slots + b0 * BUCKET_WORDS;
    const uint32_t nw = tile_words(ix, b0);
    uint64_t k[GS], v[GS];
#pragma unroll
    for (int u = 0; u < GS; ++u) {
      const uint32_t w = tile_word<TT>(u);
      v[u] = base[(w < nw ? w : 0) + SLOTS];
    }
#pragma unroll
    for (int u = 0; u < GS; ++u) {  // against the smallest sel_hi of the value's epoch
      const uint32_t w = tile_word<TT>(u);
      k[u] = KEY_EMPTY;
      if (w < nw && v[u] != VAL_UNSET && val_kind(v[u]) != HEADER && sel_hi(0, val_epoch(v[u])) <= cut.hi) k[u] = base[w];
    }
#pragma unroll
    for (int u = 0; u < GS; ++u) {
      if (!is_entry(k[u], v[u]) || !sel_leaves(k[u], sel_hi(k[u], val_epoch(v[u])), val_inst(v[u]), cut)) continue;
      base[tile_word<TT>(u)] = KEY_TOMB;
      if (val_kind(v[u]) == MEMBER) {
        const int64_t h = find_header(ix, k[u]);
        if (h < 0) {
          set_status(ix.hdr, SMETRIC_EINTERNAL);
          continue;
        }
        const uint64_t rec = val_rec(*val_ptr(ix, h));
        const uint32_t inst = val_inst(v[u]);
        atomicAnd(reinterpret_cast<unsigned long long *>(&ix.pool[rec * uint64_t(ix.words) + (inst >> 6)]),
                  ~(1ull << (inst & 63)));
      }
    }
  }
}

struct EvictWs {
  unsigned long long *count;    // the dump's entry count; EvictState
  unsigned long long *hist;     // SEL_BINS counts of a selection pass; before, the scan's counters
  uint64_t *ka, *va, *kb, *vb;  // the dump's entries and their sort ping-pong buffers; eviction: the
                                // entries in the scan's range (ka, va) and of these the last ones
                                // (kb, vb), then the entries the rebuild's tile pass leaves (ka, va)
  uint64_t *ea, *ia;            // eviction: the sample (ea); the conversion queue and deferred pairs
  void *temp;
  size_t temp_bytes;
};

size_t sort_temp_bytes(uint64_t n) {
  size_t tb = 0;
  rocprim::double_buffer<uint64_t> k(nullptr, nullptr), v(nullptr, nullptr);
  if (rocprim::radix_sort_pairs(nullptr, tb, k, v, size_t(n < 1 ? 1 : n), 0u, 64u, hipStream_t(nullptr)) != hipSuccess)
    return 0;
  return tb;
}

uint64_t evict_ws_layout(uint64_t cap, EvictWs *ws, void *base) {
  const uint64_t n = cap < 1 ? 1 : cap;
  const size_t tb = sort_temp_bytes(n);
  uint64_t off = 0;
  auto take = [&](uint64_t bytes) {
    const uint64_t o = off;
    off = round_up(off + bytes, 256);
    return o;
  };
  const uint64_t o_cnt = take(256), o_hist = take(8 * SEL_BINS), o_ka = take(8 * n), o_va = take(8 * n), o_kb = take(8 * n),
                 o_vb = take(8 * n), o_ea = take(8 * n), o_ia = take(8 * n), o_tmp = take(tb);
  if (ws) {
    char *b = static_cast<char *>(base);
    ws->count = reinterpret_cast<unsigned long long *>(b + o_cnt);
    ws->hist = reinterpret_cast<unsigned long long *>(b + o_hist);
    ws->ka = reinterpret_cast<uint64_t *>(b + o_ka);
    ws->va = reinterpret_cast<uint64_t *>(b + o_va);
    ws->kb = reinterpret_cast<uint64_t *>(b + o_kb);
    ws->vb = reinterpret_cast<uint64_t *>(b + o_vb);
    ws->ea = reinterpret_cast<uint64_t *>(b + o_ea);
    ws->ia = reinterpret_cast<uint64_t *>(b + o_ia);
    ws->temp = b + o_tmp;
    ws->temp_bytes = tb;
  }
  return off;
}

int read_hdr(const smetric_index *idx, IndexHdr *out, hipStream_t s) {
  if (hipMemcpyAsync(out, idx->hdr, sizeof(IndexHdr), hipMemcpyDeviceToHost, s) != hipSuccess) return SMETRIC_EHIP;
  return hip_rc(hipStreamSynchronize(s));
}

// The last two passes of an insert that lists its new pairs in the pair table: conversions,
// then the pairs deferred until theirs.
int ins_convert(const DevIndex &ix, const InsWs &ws, const uint32_t *session, uint32_t epoch, hipStream_t stream) {
  hipLaunchKernelGGL(spill_kernel, dim3(64), dim3(TB), 0, stream, ix, ws.trig, &ws.hdr->n_trig, &ws.hdr->abort,
                     nullptr, ws.dd, nullptr);
  hipLaunchKernelGGL(deferred_kernel, dim3(64), dim3(TB), 0, stream, ix, ws.def, &ws.hdr->n_def, &ws.hdr->abort,
                     ws.dd, session, epoch, nullptr, nullptr, nullptr);
  return hip_rc(hipGetLastError());
}

// Gather all entries and sort them by (key, instance) for the dump.  Stable LSD radix
// passes, each over the full 64-bit sort word (restricting a pass to a bit range gave
// wrong orders for some inputs with the installed rocPRIM):
//   1) by the value word (instance << 48 | epoch << 24 | session);
//   2) stably by key -- (key, instance) is unique, so this is (key, instance) order.
// On return the sorted keys/values are in (*keys_out, *vals_out).
int gather_sorted(const smetric_index *idx, const EvictWs &ws, uint64_t n, uint64_t **keys_out,
                  uint64_t **vals_out, hipStream_t s) {
  const DevIndex ix = dev_view(idx);
  int rc = fill(ws.count, 256, 0, s);
  if (rc) return rc;
  const uint64_t n_slots = ix.n_buckets * SLOTS;
  hipLaunchKernelGGL(gather_kernel, dim3(grid_for(n_slots)), dim3(TB), 0, s, ix, ws.ka, ws.va, ws.count, n);
  if ((rc = hip_rc(hipGetLastError()))) return rc;
  unsigned long long got = 0;
  if (hipMemcpyAsync(&got, ws.count, 8, hipMemcpyDeviceToHost, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
    return SMETRIC_EHIP;
  if (got != n) return SMETRIC_EINTERNAL;
  *keys_out = ws.ka;
  *vals_out = ws.va;
  if (n <= 1) return SMETRIC_OK;
  size_t tb = ws.temp_bytes;
  rocprim::double_buffer<uint64_t> vk(ws.va, ws.vb), kv(ws.ka, ws.kb);
  if (rocprim::radix_sort_pairs(ws.temp, tb, vk, kv, size_t(n), 0u, 64u, s) != hipSuccess) return SMETRIC_EHIP;
  rocprim::double_buffer<uint64_t> k2(kv.current(), kv.alternate()), v2(vk.current(), vk.alternate());
  tb = ws.temp_bytes;
  if (rocprim::radix_sort_pairs(ws.temp, tb, k2, v2, size_t(n), 0u, 64u, s) != hipSuccess) return SMETRIC_EHIP;
  *keys_out = k2.current();
  *vals_out = v2.current();
  return SMETRIC_OK;
}

}  // namespace
}  // namespace smk

using namespace smk;

extern "C" int smetric_index_bytes(uint64_t capacity, int32_t n_instances, uint64_t n_slots, uint64_t *bytes) {
  Layout L;
  if (!bytes || !layout_for(capacity, n_instances, n_slots, L)) return SMETRIC_EINVAL;
  *bytes = L.bytes;
  return SMETRIC_OK;
}

extern "C" int smetric_index_attach(smetric_index *idx, void *mem, uint64_t mem_bytes, uint64_t capacity,
                                    int32_t n_instances, uint64_t n_slots) {
  return attach(idx, mem, mem_bytes, capacity, n_instances, n_slots);
}

extern "C" int smetric_index_init(smetric_index *idx, void *mem, uint64_t mem_bytes, uint64_t capacity,
                                  int32_t n_instances, uint64_t n_slots, hipStream_t stream) {
  int rc = attach(idx, mem, mem_bytes, capacity, n_instances, n_slots);
  if (rc) return rc;
  Layout L;
  layout_for(capacity, n_instances, n_slots, L);
  if (int rc2 = fill(mem, L.bytes, 0, stream)) return rc2;
  // every slot EMPTY with an unset value
  hipLaunchKernelGGL(unset_values_kernel, dim3(grid_for(L.n_buckets)), dim3(TB), 0, stream,
                     static_cast<IndexHdr *>(idx->hdr), process_owner(), idx->slots, L.n_buckets);
  return hip_rc(hipGetLastError());
}

extern "C" int smetric_index_stats(const smetric_index *idx, uint64_t *n_entries, int32_t *status,
                                   int32_t reset_status, hipStream_t stream) {
  if (!idx || !idx->hdr) return SMETRIC_EINVAL;
  IndexHdr h;
  int rc = read_hdr(idx, &h, stream);
  if (rc) return rc;
  if (n_entries) *n_entries = h.n_entries;
  if (status) *status = h.status;
  if (reset_status) {
    hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, stream, &static_cast<IndexHdr *>(idx->hdr)->status, 0);
    if ((rc = hip_rc(hipGetLastError()))) return rc;
    rc = hip_rc(hipStreamSynchronize(stream));
  }
  return rc;
}

extern "C" int smetric_index_insert_ws_bytes(int64_t n_blocks, uint64_t *ws_bytes) {
  if (n_blocks < 0 || !ws_bytes) return SMETRIC_EINVAL;
  *ws_bytes = insert_ws_layout(n_blocks, nullptr, nullptr);
  return SMETRIC_OK;
}

extern "C" int smetric_index_insert(smetric_index *idx, const uint64_t *keys, const int64_t *blk_off,
                                    int32_t n_req, int64_t n_blocks, const int32_t *instance,
                                    const uint32_t *session, uint32_t epoch, void *workspace,
                                    uint64_t ws_bytes, hipStream_t stream) {
  if (!idx || !idx->slots || n_req < 0 || n_blocks < 0 || epoch >= EPOCH_LIMIT) return SMETRIC_EINVAL;
  if (n_req == 0) return SMETRIC_OK;
  if (!blk_off || !instance || !session || (n_blocks > 0 && !keys)) return SMETRIC_EINVAL;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) ||
      ws_bytes < insert_ws_layout(n_blocks, nullptr, nullptr))
    return SMETRIC_EWORKSPACE;
  InsWs ws;
  insert_ws_layout(n_blocks, &ws, workspace);
  const DevIndex ix = dev_view(idx);
  if (ins_small(n_blocks, n_req)) {
    hipLaunchKernelGGL(ins_small_kernel<false>, dim3(1), dim3(SI_T), 0, stream, ix, ProbeView{}, keys, blk_off, n_req,
                       n_blocks, instance, session, epoch);
    return hip_rc(hipGetLastError());
  }
  hipLaunchKernelGGL(ins_clear_kernel, dim3(grid_for(ws.n_dedupe)), dim3(TB), 0, stream, ws);
  const int per = n_blocks / n_req > 64 ? TB : 64;
  const uint64_t threads = uint64_t(n_req) * per;
  const int nt = find_threads(threads);
  const dim3 grid(find_grid(threads)), blk(nt);
  hipLaunchKernelGGL((nt == TB ? ins_probe_kernel<TB> : ins_probe_kernel<4 * TB>), grid, blk, 0, stream, ix, ws, keys,
                     blk_off, n_req, n_blocks, instance, session, epoch, per);
  hipLaunchKernelGGL((nt == TB ? ins_apply_kernel<TB> : ins_apply_kernel<4 * TB>), grid, blk, 0, stream, ix, ws, blk_off,
                     n_req, n_blocks, session, epoch, per);
  return ins_convert(ix, ws, session, epoch, stream);
}

extern "C" int smetric_index_evict_ws_bytes(const smetric_index *idx, uint64_t *ws_bytes) {
  if (!idx || !ws_bytes) return SMETRIC_EINVAL;
  *ws_bytes = evict_ws_layout(idx->capacity, nullptr, nullptr);
  return SMETRIC_OK;
}

extern "C" int smetric_index_evict(smetric_index *idx, uint32_t frac_num, uint32_t frac_den, void *workspace,
                                   uint64_t ws_bytes, hipStream_t stream) {
  if (!idx || !idx->slots || frac_den == 0 || frac_num > frac_den) return SMETRIC_EINVAL;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) ||
      ws_bytes < evict_ws_layout(idx->capacity, nullptr, nullptr))
    return SMETRIC_EWORKSPACE;
  EvictWs ws;
  evict_ws_layout(idx->capacity, &ws, workspace);
  int rc;
  if (frac_num == 0) {  // nothing leaves
    IndexHdr h;
    return read_hdr(idx, &h, stream);
  }
  const DevIndex ix = dev_view(idx);
  auto *const st = reinterpret_cast<EvictState *>(ws.count);
  static_assert(sizeof(EvictState) <= 256 && EV_LANES * EV_LINE <= SEL_BINS, "the workspace's counters");
  struct {
    union {
      EvictState st;
      char room[256];
    };
    unsigned long long counts[EV_LANES * EV_LINE];  // as the workspace holds them
  } seen;
  static_assert(sizeof(seen) == 256 + 8 * EV_LANES * EV_LINE, "the state and the counters are one run of it");
  const uint64_t n_tiles = (ix.n_buckets + TILE - 1) / TILE;
  // a sample pays from 2^15 buckets on (a scan there copies at most 4 MB); it needs its room
  const bool sampled = ix.n_buckets >= (uint64_t(1) << 15) && idx->capacity >= uint64_t(EV_SAMPLE) * SLOTS;
  uint64_t n = 0, m = 0, live = 0, n_tomb = 0, below = 0, inside = 0;
  for (int round = sampled ? 0 : 1; round < 2; ++round) {  // second: the range missed the cut, take everything
    hipLaunchKernelGGL(evict_sample_kernel, dim3(round == 0 ? EV_SAMPLE * SLOTS / TB : 1), dim3(TB), 0, stream, ix, st,
                       ws.hist, round == 0 ? ws.ea : nullptr);
    if (round == 0)
      hipLaunchKernelGGL(evict_range_kernel, dim3(1), dim3(FIN_T), 0, stream, ws.ea, frac_num, frac_den, st);
    hipLaunchKernelGGL(evict_scan_kernel, dim3(n_tiles < 1024 ? n_tiles : 1024), dim3(TB), 0, stream, ix, st, ws.hist,
                       ws.ka, ws.va, idx->capacity);
    if ((rc = hip_rc(hipGetLastError()))) return rc;
    if (hipMemcpyAsync(&seen, ws.count, sizeof(seen), hipMemcpyDeviceToHost, stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
      return SMETRIC_EHIP;
    n = seen.st.n_entries;
    m = uint64_t((static_cast<unsigned __int128>(n) * frac_num + frac_den - 1) / frac_den);
    if (m == 0) return SMETRIC_OK;
    inside = seen.st.n_in;
    live = n_tomb = below = 0;
    for (int b = 0; b < EV_LANES; ++b) {
      live += seen.counts[b * EV_LINE];
      n_tomb += seen.counts[b * EV_LINE + 1];
      below += seen.counts[b * EV_LINE + 2];
    }
    if (live != n || n > idx->capacity) return SMETRIC_EINTERNAL;
    if (below < m && m <= below + inside) break;
  }
  if (below >= m || m > below + inside) return SMETRIC_EINTERNAL;
  // select the m-th smallest among the entries in the range: first the digits that its two
  // ends share, then one digit per pass; stop once a whole bin is evicted
  SelPrefix p{};
  uint64_t rem = m - below, on_prefix = inside;  // rank (1-based) among the entries on the prefix
  for (int l = 0; l < 5; ++l) {                  // the digits that sel_hi holds whole
    const uint64_t lo = seen.st.lo, hi = seen.st.hi;
    const uint32_t d = sel_digit(lo << 24, (lo >> 40) << 24, l);
    if (hi >> 62 || d != sel_digit(hi << 24, (hi >> 40) << 24, l)) break;
    p.digit[l] = d;
    p.level = l + 1;
  }
  const SelCut *cut_dev = nullptr;  // the cut, once a kernel decides it
  uint64_t *sk = ws.ka, *sv = ws.va;
  while (p.level < SEL_LEVELS && rem < on_prefix) {
    const int grid = grid_for(inside) < 1024 ? grid_for(inside) : 1024;
    if (on_prefix <= SEL_FIN) {  // few left: copied out if they are spread over more, and the rest without the host
      const bool copy = inside > SEL_FIN;
      if (copy)
        hipLaunchKernelGGL(sel_copy_kernel, dim3(grid), dim3(TB), 0, stream, sk, sv, inside, p, &st->n_fin, ws.kb,
                           ws.vb, idx->capacity);
      hipLaunchKernelGGL(sel_finish_kernel, dim3(1), dim3(FIN_T), 0, stream, ix, copy ? ws.kb : sk, copy ? ws.vb : sv,
                         copy ? on_prefix : inside, p, rem, on_prefix, copy ? &st->n_fin : nullptr, st);
      cut_dev = &st->cut;
      break;
    }
    unsigned long long hh[SEL_BINS];
    if ((rc = fill(ws.hist, sizeof(hh), 0, stream))) return rc;
    hipLaunchKernelGGL(sel_hist_kernel, dim3(grid), dim3(TB), 0, stream, sk, sv, inside, p, ws.hist);
    if (hipMemcpyAsync(hh, ws.hist, sizeof(hh), hipMemcpyDeviceToHost, stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
      return SMETRIC_EHIP;
    uint64_t sum = 0;
    int b = 0;
    while (b < SEL_BINS && sum + hh[b] < rem) sum += hh[b++];
    if (b == SEL_BINS) return SMETRIC_EINTERNAL;
    p.digit[p.level++] = uint32_t(b);
    rem -= sum;
    on_prefix = hh[b];  // rem == on_prefix: the whole bin goes, the prefix itself is the cut
  }
  if (rem < on_prefix && !cut_dev) return SMETRIC_EINTERNAL;  // the full tuple is unique
  const SelCut cut = sel_cut(p, seen.st.hi);
  // few tombstones: evict in place, the survivors keep their slots.  Tombstones may take
  // an eighth of the slots, and at most half of what stays free with the live entries at
  // capacity (the same eighth under the default 3/4 sizing), so every chain keeps
  // reaching an EMPTY slot
  const uint64_t n_slots = ix.n_buckets * SLOTS;
  const uint64_t reserved = idx->capacity + uint64_t(ix.threshold) * ix.n_records;
  const uint64_t tomb_cap_free = n_slots > reserved ? (n_slots - reserved) / 2 : 0;
  const uint64_t tomb_cap = tomb_cap_free < n_slots / 8 ? tomb_cap_free : n_slots / 8;
  if (n_tomb + m <= tomb_cap) {
    hipLaunchKernelGGL(evict_tomb_kernel, dim3(n_tiles < MAX_GRID ? n_tiles : MAX_GRID), dim3(TT), 0, stream, ix, cut,
                       cut_dev, (unsigned long long)(n - m));
    if ((rc = hip_rc(hipGetLastError()))) return rc;
    return hip_rc(hipStreamSynchronize(stream));
  }
  // else rebuild from the survivors (the entries above the cut, exactly n - m of them),
  // which also clears every tombstone: the tile pass (writes every bucket: no clear needed),
  // then the claims for what it left
  if ((rc = fill(ix.pool, ix.n_records * uint64_t(ix.words) * 8, 0, stream))) return rc;
  hipLaunchKernelGGL(rebuild_tile_kernel, dim3(n_tiles), dim3(TILE), 0, stream, ix, cut, cut_dev, ws.ka, ws.va,
                     &st->n_left, idx->capacity, (unsigned long long)(n - m));
  hipLaunchKernelGGL(rebuild_claim_kernel, dim3(n_tiles < CLAIM_WG ? n_tiles : CLAIM_WG), dim3(TB), 0, stream, ix,
                     ws.ka, ws.va, &st->n_left, ws.ea, &st->n_trig, ws.ia, &st->n_def, idx->capacity);
  hipLaunchKernelGGL(spill_kernel, dim3(64), dim3(TB), 0, stream, ix, ws.ea, &st->n_trig, nullptr, ws.ka, nullptr,
                     nullptr);
  // every member of a key with a bitmap record is deferred here (millions): the full grid
  hipLaunchKernelGGL(deferred_kernel, dim3(MAX_GRID), dim3(TB), 0, stream, ix, ws.ia, &st->n_def, nullptr, nullptr,
                     nullptr, 0u, ws.ka, ws.va, nullptr);
  if ((rc = hip_rc(hipGetLastError()))) return rc;
  return hip_rc(hipStreamSynchronize(stream));
}

extern "C" int smetric_index_dump(const smetric_index *idx, uint64_t *keys_out, uint64_t *vals_out, uint64_t cap,
                                  void *workspace, uint64_t ws_bytes, uint64_t *n_out, hipStream_t stream) {
  if (!idx || !idx->slots || !n_out || (cap > 0 && (!keys_out || !vals_out))) return SMETRIC_EINVAL;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) ||
      ws_bytes < evict_ws_layout(idx->capacity, nullptr, nullptr))
    return SMETRIC_EWORKSPACE;
  EvictWs ws;
  evict_ws_layout(idx->capacity, &ws, workspace);
  IndexHdr h;
  int rc = read_hdr(idx, &h, stream);
  if (rc) return rc;
  const uint64_t n = h.n_entries;
  *n_out = n;
  if (n == 0) return SMETRIC_OK;
  uint64_t *keys, *vals;
  if ((rc = gather_sorted(idx, ws, n, &keys, &vals, stream))) return rc;
  const uint64_t c = n < cap ? n : cap;
  if (c) {
    if (hipMemcpyAsync(keys_out, keys, 8 * c, hipMemcpyDeviceToDevice, stream) != hipSuccess ||
        hipMemcpyAsync(vals_out, vals, 8 * c, hipMemcpyDeviceToDevice, stream) != hipSuccess)
      return SMETRIC_EHIP;
  }
  return hip_rc(hipStreamSynchronize(stream));
}

extern "C" int smetric_index_insert_probed(smetric_index *idx, const void *probe, uint64_t probe_bytes,
                                           int32_t n_req, int64_t n_blocks, const int32_t *instance,
                                           const uint32_t *session, uint32_t epoch, void *workspace,
                                           uint64_t ws_bytes, hipStream_t stream) {
  if (!idx || !idx->slots || n_req < 0 || n_blocks < 0 || n_blocks >= (int64_t(1) << 31) || epoch >= EPOCH_LIMIT)
    return SMETRIC_EINVAL;
  if (n_req == 0) return SMETRIC_OK;
  if (!instance || !session) return SMETRIC_EINVAL;
  if (!probe || (reinterpret_cast<uintptr_t>(probe) & 255) || probe_bytes < probe_layout(n_blocks, nullptr, nullptr))
    return SMETRIC_EWORKSPACE;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) ||
      ws_bytes < insert_ws_layout(n_blocks, nullptr, nullptr))
    return SMETRIC_EWORKSPACE;
  ProbeView pv;
  probe_layout(n_blocks, &pv, const_cast<void *>(probe));
  InsWs ws;
  insert_ws_layout(n_blocks, &ws, workspace);
  const DevIndex ix = dev_view(idx);
  if (n_blocks <= SI_MAX) {
    hipLaunchKernelGGL(ins_small_kernel<true>, dim3(1), dim3(SI_T), 0, stream, ix, pv, nullptr, nullptr, n_req, n_blocks,
                       instance, session, epoch);
    return hip_rc(hipGetLastError());
  }
  if (direct_batch(uint64_t(n_blocks))) {
    hipLaunchKernelGGL(ins_clear_kernel, dim3(grid_for(ws.n_dedupe)), dim3(TB), 0, stream, ws);
    const int nt = find_threads(uint64_t(n_blocks));
    const dim3 grid(find_grid(uint64_t(n_blocks))), blk(nt);
    hipLaunchKernelGGL((nt == TB ? insd_find_kernel<TB> : insd_find_kernel<4 * TB>), grid, blk, 0, stream, ix, pv, ws,
                       n_blocks, instance, session, epoch);
    hipLaunchKernelGGL((nt == TB ? ins_apply_kernel<TB> : ins_apply_kernel<4 * TB>), grid, blk, 0, stream, ix, ws, nullptr,
                       n_req, n_blocks, session, epoch, TB);
    return ins_convert(ix, ws, session, epoch, stream);
  }
  const dim3 blk(TB), chunks(NREG * KCH);
  hipLaunchKernelGGL(insp_head_kernel, dim3(HEAD_WG), blk, 0, stream, ix, ws, instance, session, n_req);
  hipLaunchKernelGGL(insp_classify_kernel, dim3(INS_WG), blk, 0, stream, ix, pv, ws, instance, session, epoch);
  hipLaunchKernelGGL(insp_bcount_kernel, chunks, blk, 0, stream, ix, ws);
  hipLaunchKernelGGL(insp_bscan_kernel, dim3(NREG), dim3(SCAN_T), 0, stream, ws);
  hipLaunchKernelGGL(insp_bscatter_kernel, chunks, blk, 0, stream, ix, ws);
  hipLaunchKernelGGL(insp_bdedupe_kernel, dim3(DEDUPE_WG), dim3(DD_T), 0, stream, ix, ws);
  hipLaunchKernelGGL(insp_place_kernel, dim3(PLACE_WG), blk, 0, stream, ix, pv, ws, session, epoch);
  hipLaunchKernelGGL(spill_kernel, dim3(64), blk, 0, stream, ix, ws.trig, &ws.hdr->n_trig, &ws.hdr->abort,
                     nullptr, nullptr, ws.np);
  hipLaunchKernelGGL(deferred_kernel, dim3(64), blk, 0, stream, ix, ws.def, &ws.hdr->n_def, &ws.hdr->abort,
                     ws.dd, session, epoch, nullptr, nullptr, ws.np);
  return hip_rc(hipGetLastError());
}
