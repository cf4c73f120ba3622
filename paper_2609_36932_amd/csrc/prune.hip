// Maximizing Differential Advantage Pruning (Sec. 3.2; Alg. 1 Phase 2), the keep-ratio
// budget, and stream compaction of kept tokens.  Every decision is integer or exact:
//   K1 ngram_set    one block per trajectory: pack n-grams into keys (21 bits per token) and list
//                   the distinct ones through a set in LDS (bits for n = 1, else hashed).  Also
//                   writes which question owns each trajectory.
//   K2 pair_conflict one block per trajectory i: |N_n(o_i) & N_n(o_j)| for every j < i of its
//                   question and class, by looking the keys of j up in a set of i in LDS, then
//                   theta < tau as  tau_den * (|U| - |I|) < tau_num * |U|  in int64; the
//                   outcomes are trajectory i's row of conflict bits.
//   K0 group_eps    (continuous rewards, appendix on the grounding task) one wavefront per
//                   question: classes = connected components of |A_i - A_j| < eps, from the
//                   sorted advantages (a new class wherever a gap is >= eps).
//   K3 select       one wavefront per question: the greedy independent set in visiting
//                   order (|A| descending, ties by index, when advantages are given; else
//                   ascending index), then the budget as "keep the K smallest (tier, rank,
//                   class position) keys" -- the same list a class round-robin produces.
//   K3b dp_fill     (optional) Alg. 1's DP alignment of the kept count, one block.
//   K4 compaction   exclusive scans of kept flags and kept lengths and a coalesced fill of
//                   tok_src, one block per trajectory (over 4096 trajectories: the scans in a
//                   one-block launch of their own).
#include <type_traits>

#include "common.h"

namespace fastrl {

#define FR_TRY(x)                     \
  do {                                \
    int rc_ = (x);                    \
    if (rc_ != FASTRL_OK) return rc_; \
  } while (0)

constexpr int kMaxGroupPrune = 256;
constexpr int kMaxLenPrune = 16384;
constexpr int kConflictWords = kMaxGroupPrune / 64;

// ---- sets of n-gram keys in LDS
// n = 1 with a vocabulary up to kMaxBitVocab: one bit per token id.  One LDS access per key and no
// probing, so lookups of several keys overlap (19 KB at V = 152064).
constexpr int kMaxBitVocab = 1 << 19;  // 64 KB
struct BitSet {
  typedef uint32_t Key;
  static constexpr Key kNone = 0xffffffffu;
  // 32-bit words of the set (m: keys to insert), in 16-byte pieces
  static __host__ __device__ int words(int V, int m) { return ((V + 127) / 128) * 4; }
  static constexpr uint32_t kClear = 0u;
  uint32_t* w;
  __device__ BitSet(char* lds, int V, int m) : w(reinterpret_cast<uint32_t*>(lds)) {}
  // true if `key` was not in the set (a plain read first: head-heavy ids are mostly there already,
  // and their atomics on one address would run one by one)
  __device__ __forceinline__ bool insert(Key key) {
    const uint32_t bit = 1u << (key & 31);
    if (reinterpret_cast<volatile uint32_t*>(w)[key >> 5] & bit) return false;
    return (atomicOr(&w[key >> 5], bit) & bit) == 0;
  }
  // an insert of a key that no other thread inserts
  __device__ __forceinline__ void insert_new(Key key) { atomicOr(&w[key >> 5], 1u << (key & 31)); }
  // how many of the U keys (kNone: no key) are in the set
  template <int U>
  __device__ __forceinline__ int count(const Key (&k)[U]) const {
    int n = 0;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k[u] != kNone) n += (w[k[u] >> 5] >> (k[u] & 31)) & 1u;
    return n;
  }
};
// otherwise a hash set: open addressing, linear probing, of whose slots at least a sixth stay empty
// (so every probe ends).  No key equals the empty marker: three 21-bit ids fill 63 bits.  A wavefront
// waits for the longest of its probes, so sets of up to 32 KB take four slots a key: with two, the
// pair tests of 8192 rollouts of 254 trigrams took 158 us in place of 88 (blocks of 512).
struct HashSet {
  typedef uint64_t Key;
  static constexpr Key kNone = ~0ull;
  // half of the slots empty where the LDS allows it; 156 KB: 16384 keys leave 3584 slots empty
  static constexpr int kMaxSlots = 19968;
  static constexpr int kSmallSlots = 4096;  // 32 KB
  static __host__ __device__ int slots(int m) {
    const int s = 4 * m < kSmallSlots ? 4 * m : 2 * m < kSmallSlots ? kSmallSlots : 2 * m;
    return s < 64 ? 64 : s < kMaxSlots ? s : kMaxSlots;
  }
  static __host__ __device__ int words(int V, int m) { return slots(m) * 2; }
  static constexpr uint32_t kClear = 0xffffffffu;
  uint64_t* tab;
  uint32_t size;
  __device__ HashSet(char* lds, int V, int m)
      : tab(reinterpret_cast<uint64_t*>(lds)), size(uint32_t(slots(m))) {}
  __device__ __forceinline__ uint32_t slot(Key k) const {
    return __umulhi(uint32_t((k * 0x9e3779b97f4a7c15ull) >> 32), size);
  }
  __device__ __forceinline__ bool insert(Key key) {
    uint32_t h = slot(key);
    for (;;) {
      Key c = reinterpret_cast<volatile Key*>(tab)[h];
      if (c == kNone) {
        c = atomicCAS(reinterpret_cast<unsigned long long*>(tab + h), (unsigned long long)kNone,
                      (unsigned long long)key);
        if (c == kNone) return true;
      }
      if (c == key) return false;
      if (++h == size) h = 0;
    }
  }
  __device__ __forceinline__ void insert_new(Key key) {
    uint32_t h = slot(key);
    while (atomicCAS(reinterpret_cast<unsigned long long*>(tab + h), (unsigned long long)kNone,
                     (unsigned long long)key) != kNone)
      if (++h == size) h = 0;
  }
  // (the U probes of a round are in flight together)
  template <int U>
  __device__ __forceinline__ int count(const Key (&k)[U]) const {
    uint32_t h[U];
    bool open[U], any = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      h[u] = slot(k[u]);
      open[u] = k[u] != kNone;
      any |= open[u];
    }
    int n = 0;
    while (any) {
      Key c[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (open[u]) c[u] = tab[h[u]];
      any = false;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        n += open[u] && c[u] == k[u];
        open[u] = open[u] && c[u] != k[u] && c[u] != kNone;
        if (++h[u] == size) h[u] = 0;
        any |= open[u];
      }
    }
    return n;
  }
};
// empties a set (its words are a multiple of 4 and at most 16-byte aligned pieces)
template <typename S>
__device__ __forceinline__ void set_clear(char* lds, int V, int m, int tid, int threads) {
  const uint32_t c = S::kClear;
  uint4* p = reinterpret_cast<uint4*>(lds);
  for (int j = tid; j < S::words(V, m) / 4; j += threads) p[j] = make_uint4(c, c, c, c);
}
// whether a question's members can be pruned (K3 flags the others)
__device__ __forceinline__ bool group_ok(int g0, int g1, int N, int max_group) {
  return g0 >= 0 && g1 >= g0 && g1 <= N && g1 - g0 <= max_group;
}
// a trajectory's list of distinct keys: at its first token's place in the key array
template <typename K>
__device__ __forceinline__ K* key_list(uint64_t* keys, int64_t first) {
  return reinterpret_cast<K*>(keys + first);
}

// ---------------------------------------------------------------------------- K1
// Distinct n-grams of each trajectory, in any order (only set sizes and memberships are used).
// Bound by latency: a few dependent LDS accesses per key.  1538 trajectories of 256-2048 tokens:
// 78 us as a bitonic sort of P = 2048 keys per block (66 passes over LDS), 11 us as a bit set.
template <typename S>
__global__ __launch_bounds__(256) void ngram_set_kernel(
    const int32_t* __restrict__ tokens, const int64_t* __restrict__ toff, int64_t T_total,
    int32_t V, int32_t n, int32_t max_len, uint64_t* __restrict__ keys,
    int32_t* __restrict__ nuniq, const int32_t* __restrict__ group_off, int32_t Q, int32_t N,
    int32_t max_group, int2* __restrict__ owner, int32_t* __restrict__ status) {
  typedef typename S::Key K;
  extern __shared__ __attribute__((aligned(16))) char set_raw[];
  __shared__ int32_t count, bad_flag;
  const int i = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  // the last wavefront notes the owner of the members of question i (and i + gridDim.x, ..)
  if (tid >= 192)
    for (int64_t q = i; q < Q; q += gridDim.x) {
      const int g0 = group_off[q], g1 = group_off[q + 1];
      if (!group_ok(g0, g1, N, max_group)) continue;  // flagged by K3
      for (int t = g0 + lane; t < g1; t += 64) owner[t] = make_int2(int(q), g0);
    }
  const int64_t a = toff[i], b = toff[i + 1];
  const bool off_ok = a >= 0 && b >= a && b <= T_total;
  if (!off_ok || b - a > max_len) {
    if (tid == 0) {
      set_status(status, off_ok ? FASTRL_SB_SEQ_TOO_LONG : FASTRL_SB_BAD_OFFSETS);
      nuniq[i] = 0;
    }
    return;
  }
  const int L = int(b - a);
  const int m = L >= n ? L - n + 1 : 0;
  S set(set_raw, V, m);
  if (tid == 0) count = bad_flag = 0;
  if (m > 0) set_clear<S>(set_raw, V, m, tid, 256);
  __syncthreads();
  K* out = key_list<K>(keys, a);
  for (int j0 = 0; j0 < m; j0 += 256) {
    const int j = j0 + tid;
    bool fresh = false;
    K key = 0;
    if (j < m) {
      for (int k = 0; k < n; ++k) {
        int32_t t = tokens[a + j + k];
        if (t < 0 || t >= V) {
          bad_flag = 1;
          t = 0;
        }
        key |= K(uint32_t(t)) << (21 * k);
      }
      fresh = set.insert(key);
    }
    const uint64_t mask = __ballot(fresh);
    if (mask) {
      int base = 0;
      if (lane == 0) base = atomicAdd(&count, __popcll(mask));
      base = __builtin_amdgcn_readfirstlane(base);
      if (fresh) out[base + __popcll(mask & ((1ull << lane) - 1))] = key;
    }
  }
  __syncthreads();
  if (tid == 0) {
    nuniq[i] = count;
    if (bad_flag) set_status(status, FASTRL_SB_BAD_TOKEN);
  }
}

// ---------------------------------------------------------------------------- K0
// Continuous-reward classes of one question: the connected components of the relation
// |A_i - A_j| < eps over its float32 advantages (read as float64, gaps in float64),
// numbered by lowest member index.  Sorting by (A, index) puts every component on a run of
// consecutive positions, and a run ends where the gap to the next value is >= eps.
__global__ __launch_bounds__(64) void group_eps_kernel(
    const float* __restrict__ adv, const int32_t* __restrict__ group_off, int32_t N,
    int32_t max_group, double eps, int32_t* __restrict__ cls_out, int32_t* __restrict__ status) {
  __shared__ float a[kMaxGroupPrune];
  __shared__ int32_t sidx[kMaxGroupPrune];   // position -> member
  __shared__ int32_t comp[kMaxGroupPrune];   // member -> component (in sorted order)
  __shared__ int32_t label[kMaxGroupPrune];  // component -> class id
  const int q = blockIdx.x;
  const int lane = threadIdx.x;
  const int g0 = group_off[q], g1 = group_off[q + 1];
  if (g0 < 0 || g1 < g0 || g1 > N || g1 - g0 > max_group) return;  // flagged by K3
  const int G = g1 - g0;
  int bad = 0;
  for (int i = lane; i < G; i += 64) {
    float v = adv[g0 + i];
    if (!isfinite(v)) {  // keeps the ranks a permutation
      bad = 1;
      v = 0.0f;
    }
    a[i] = v;
  }
  if (bad) set_status(status, FASTRL_SB_BAD_REWARD);
  __syncthreads();
  for (int i = lane; i < G; i += 64) {
    const float ai = a[i];
    int r = 0;
    for (int j = 0; j < G; ++j) r += (a[j] < ai) || (a[j] == ai && j < i);
    sidx[r] = i;
  }
  __syncthreads();
  if (lane == 0 && G > 0) {
    int c = 0;
    comp[sidx[0]] = 0;
    for (int p = 1; p < G; ++p) {
      if (__dsub_rn(double(a[sidx[p]]), double(a[sidx[p - 1]])) >= eps) ++c;
      comp[sidx[p]] = c;
    }
    for (int k = 0; k <= c; ++k) label[k] = -1;
    int next = 0;
    for (int i = 0; i < G; ++i) {
      const int k = comp[i];
      if (label[k] < 0) label[k] = next++;
      cls_out[g0 + i] = label[k];
    }
  }
}

// ---------------------------------------------------------------------------- K2
// Conflict row of trajectory t0 + blockIdx.x, member i of its question: bit j (j < i, same class) is
// set where theta < tau.  The set of i is built once in LDS and each wavefront looks up the keys of
// every eighth candidate j, 512 at a time (coalesced reads of j's list, all in flight together; one
// LDS read per key in a bit set).  Bound by the latency of those reads.  128 questions of 8-16
// rollouts of 256-2048 tokens: 477 us with one block per question and binary searches in global
// memory, 15 us so (unigrams).  One block per trajectory and not per (question, max_group) slot: the
// launch follows the rollouts there are, whatever bound the caller states for their groups (1024
// questions of 8 under max_group = 256: 593 us by slot, 131 us so; under max_group = 8 level).
// Threads (launch_sets): with few blocks, or many candidates each, the wavefronts of one work on its
// candidates at once; from 4096 blocks on the chip is full, and a short list of few candidates
// occupies a wavefront or two of a block, whose others only keep blocks out.  Pair tests in us, hashed
// trigrams, 128 / 256 / 512 threads: 8192 rollouts of 254 35 / 38 / 53 (1024 questions of 8), 16384 of
// 62 22 / 39 / 69 (4096 of 4), 8192 of 698 139 / 100 / 108, 2048 of 698 81 / 53 / 47, 8192 of 1499
// 471 / 320 / 259; unigrams, 256 / 512: 8192 of 256 20 / 29, 2048 of 256 in groups of 128 46 / 28.
// (Binary searches in sorted lists, one block per question, took 53, 13 and 195 us in the first three,
// after sorts of 48, 52 and 151 us where the sets take 21, 22 and 41.)
// U: keys that a lane looks up at a time.  Hashed, each key of the U waits for the slowest: up to 512
// keys 2 (16384 rollouts of 62: 22 us, 28 with 4, 46 with 8), above 4 (8 loses 20-30%).
// most blocks of one pair launch (a launch's threads number below 2^32)
constexpr int kPairBlocks = 1 << 22;
template <typename S, int THREADS, int U>
__global__ __launch_bounds__(THREADS) void pair_conflict_kernel(
    const int64_t* __restrict__ toff, const int32_t* __restrict__ group_off,
    const int32_t* __restrict__ class_id, uint64_t* __restrict__ keys,
    const int32_t* __restrict__ nuniq, const int2* __restrict__ owner, int32_t t0, int32_t Q,
    int32_t N, int32_t V, int32_t max_group, int32_t tau_num, int32_t tau_den,
    uint64_t* __restrict__ conflict) {
  typedef typename S::Key K;
  extern __shared__ __attribute__((aligned(16))) char set_raw[];
  __shared__ int32_t cand[kMaxGroupPrune];
  __shared__ unsigned long long row[kConflictWords];
  const int t = t0 + blockIdx.x;
  // a trajectory of no valid question has an owner that K1 did not write: these tests keep the reads
  // in range, and the one below refuses it (its loads go out with the candidates')
  const int2 o = owner[t];
  const int q = o.x, g0 = o.y;
  if (q < 0 || q >= Q || g0 < 0 || g0 > t || t - g0 >= max_group) return;
  const int i = t - g0;
  const int q0 = group_off[q], q1 = group_off[q + 1];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int words = (max_group + 63) / 64;
  const int cls = class_id[t], na = nuniq[t];
  // candidates j < i, listed by every wavefront alike (same values to the same places)
  int nc = 0;
  for (int j0 = 0; j0 < i; j0 += 64) {
    const bool c = j0 + lane < i && class_id[g0 + j0 + lane] == cls;
    const uint64_t mask = __ballot(c);
    if (c) cand[nc + __popcll(mask & ((1ull << lane) - 1))] = j0 + lane;
    nc += __popcll(mask);
  }
  if (q0 != g0 || t >= q1 || !group_ok(q0, q1, N, max_group)) return;
  if (tid < kConflictWords) row[tid] = 0;
  S set(set_raw, V, na);
  if (nc > 0 && na > 0) {
    const K* ka = key_list<K>(keys, toff[t]);
    set_clear<S>(set_raw, V, na, tid, THREADS);
    __syncthreads();
    for (int e = tid; e < na; e += THREADS) set.insert_new(ka[e]);
  }
  __syncthreads();
  for (int p = wv; p < nc; p += THREADS / 64) {
    const int j = cand[p];
    const int nb = nuniq[g0 + j];
    int cnt = 0;
    if (na > 0 && nb > 0) {
      const K* kb = key_list<K>(keys, toff[g0 + j]);
      for (int e0 = 0; e0 < nb; e0 += 64 * U) {
        K k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int e = e0 + 64 * u + lane;
          k[u] = e < nb ? kb[e] : S::kNone;
        }
        cnt += set.template count<U>(k);
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    if (lane == 0) {
      const int64_t both = cnt, any = int64_t(na) + nb - cnt;
      bool c;
      if (any == 0) c = tau_num > 0;  // theta = 0 for two empty sets
      else c = int64_t(tau_den) * (any - both) < int64_t(tau_num) * any;
      if (c) atomicOr(&row[j >> 6], 1ull << (j & 63));
    }
  }
  __syncthreads();
  if (tid < words) conflict[size_t(t) * words + tid] = row[tid];
}

// ---------------------------------------------------------------------------- K3
__global__ __launch_bounds__(64) void select_kernel(
    const float* __restrict__ rewards, const int32_t* __restrict__ group_off,
    const int32_t* __restrict__ class_id, const float* __restrict__ adv,
    const uint8_t* __restrict__ group_valid, int32_t N, int32_t max_group, double keep_ratio,
    const uint64_t* __restrict__ conflict, const int2* __restrict__ owner,
    uint8_t* __restrict__ keep_mask, int32_t* __restrict__ mdap_count,
    int32_t* __restrict__ class_out, int32_t* __restrict__ status) {
  __shared__ uint64_t crow[kMaxGroupPrune][kConflictWords];  // conflict row of member i
  __shared__ float rew[kMaxGroupPrune];
  __shared__ uint8_t mdap[kMaxGroupPrune];
  __shared__ int32_t cls[kMaxGroupPrune];
  __shared__ int32_t vpos[kMaxGroupPrune];     // visiting position of member i
  __shared__ int32_t ord[kMaxGroupPrune];      // member at visiting position p
  __shared__ float aabs[kMaxGroupPrune];
  __shared__ int32_t crep[kMaxGroupPrune];     // first visited member of class c
  __shared__ int32_t cmin[kMaxGroupPrune];     // lowest member index of class c
  __shared__ double kappa[kMaxGroupPrune];     // kappa of class c
  __shared__ int32_t cpos[kMaxGroupPrune];     // rank of class c in the budget order
  __shared__ int32_t rank[kMaxGroupPrune];     // rank of member i inside its class tier
  const int q = blockIdx.x;
  const int lane = threadIdx.x;
  const int g0 = group_off[q], g1 = group_off[q + 1];
  if (g0 < 0 || g1 < g0 || g1 > N) {
    if (lane == 0) {
      set_status(status, FASTRL_SB_BAD_OFFSETS);
      mdap_count[q] = 0;
    }
    return;
  }
  const int G = g1 - g0;
  if (G > max_group) {
    for (int i = lane; i < G; i += 64) keep_mask[g0 + i] = 0;
    if (lane == 0) {
      set_status(status, FASTRL_SB_GROUP_TOO_BIG);
      mdap_count[q] = 0;
    }
    return;
  }
  for (int i = lane; i < G; i += 64) {
    int c = class_id[g0 + i];
    if (c < 0 || c >= G) {  // class ids are 0..G-1
      set_status(status, FASTRL_SB_BAD_INDEX);
      c = 0;
    }
    cls[i] = c;
    if (class_out) class_out[g0 + i] = c;
  }
  const bool valid = group_valid ? group_valid[q] != 0 : true;
  if (!valid || G == 0) {
    for (int i = lane; i < G; i += 64) keep_mask[g0 + i] = 0;
    if (lane == 0) mdap_count[q] = 0;
    return;
  }
  // visiting order: |A| descending, ties by index (Alg. 1); ascending index without A
  if (adv) {
    for (int i = lane; i < G; i += 64) {
      const float v = adv[g0 + i];
      aabs[i] = isfinite(v) ? fabsf(v) : 0.0f;  // non-finite A was flagged upstream
    }
    __syncthreads();
    for (int i = lane; i < G; i += 64) {
      const float ai = aabs[i];
      int r = 0;
      for (int j = 0; j < G; ++j) r += (aabs[j] > ai) || (aabs[j] == ai && j < i);
      vpos[i] = r;
      ord[r] = i;
    }
  } else {
    for (int i = lane; i < G; i += 64) {
      vpos[i] = i;
      ord[i] = i;
    }
  }
  __syncthreads();
  const int words = (max_group + 63) / 64;
  // (offsets that are not monotone can give a trajectory to two questions: they are flagged, and
  // its row belongs to the one that K1 noted)
  const uint64_t* cq = conflict + size_t(g0) * words;
  for (int e = lane; e < G * kConflictWords; e += 64) {
    const int i = e / kConflictWords, w = e % kConflictWords;
    const int own = owner[g0 + i].x;
    const uint64_t c = cq[i * words + min(w, words - 1)];  // (both loads before the test)
    crow[i][w] = w < words && own == q ? c : 0;
  }
  for (int i = lane; i < G; i += 64) rew[i] = rewards[g0 + i];
  __syncthreads();
  // greedy maximal independent set per class, members in visiting order: lane l holds the whole
  // conflict row (earlier and later members) of the members at positions l, l + 64, ..; the kept
  // set is the same in every lane
  uint64_t kept[kConflictWords] = {};
  int count = 0;
#pragma unroll
  for (int pb = 0; pb < kConflictWords; ++pb) {
    if (pb * 64 >= G) break;
    const int pos = pb * 64 + lane;
    const int me = pos < G ? ord[pos] : 0;
    uint64_t full[kConflictWords];
#pragma unroll
    for (int w = 0; w < kConflictWords; ++w) full[w] = pos < G ? crow[me][w] : 0;
    for (int j = 0; j < G; ++j) {
      const uint64_t bit = (crow[j][me >> 6] >> (me & 63)) & 1ull;
#pragma unroll
      for (int w = 0; w < kConflictWords; ++w)
        if ((j >> 6) == w) full[w] |= bit << (j & 63);
    }
    const int np = min(64, G - pb * 64);
    for (int p = 0; p < np; ++p) {
      const int i = __builtin_amdgcn_readlane(me, p);
      uint64_t hit = 0;
#pragma unroll
      for (int w = 0; w < kConflictWords; ++w) {
        if (w * 64 >= G) break;
        const uint64_t f = uint64_t(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(full[w])), p))) |
                           uint64_t(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(full[w] >> 32)), p))) << 32;
        hit |= f & kept[w];
      }
      if (hit == 0) {
#pragma unroll
        for (int w = 0; w < kConflictWords; ++w)
          if ((i >> 6) == w) kept[w] |= 1ull << (i & 63);
        ++count;
      }
    }
  }
  for (int i = lane; i < G; i += 64) {
    uint64_t k = 0;
#pragma unroll
    for (int w = 0; w < kConflictWords; ++w)
      if ((i >> 6) == w) k = kept[w];
    mdap[i] = uint8_t((k >> (i & 63)) & 1ull);
  }
  if (lane == 0) mdap_count[q] = count;
  __syncthreads();
  if (!(keep_ratio > 0.0)) {
    for (int i = lane; i < G; i += 64) keep_mask[g0 + i] = mdap[i];
    return;
  }
  // budget: kappa_k = |G r_k - sum_j r_j| (sum in index order, float64; r_k the reward of
  // the class's first visited member); classes ordered by kappa descending, then by their
  // lowest member index
  double total = 0.0;
  for (int j = 0; j < G; ++j) total = __dadd_rn(total, double(rew[j]));
  for (int c = lane; c < G; c += 64) {
    int rep = -1, low = -1;
    for (int j = G - 1; j >= 0; --j) {
      if (cls[ord[j]] == c) rep = ord[j];
      if (cls[j] == c) low = j;
    }
    crep[c] = rep;
    cmin[c] = low;
    if (rep >= 0) kappa[c] = fabs(__dsub_rn(__dmul_rn(double(G), double(rew[rep])), total));
  }
  __syncthreads();
  for (int c = lane; c < G; c += 64) {
    if (crep[c] < 0) continue;
    int pos = 0;
    for (int e = 0; e < G; ++e) {
      if (crep[e] < 0 || e == c) continue;
      if (kappa[e] > kappa[c] || (kappa[e] == kappa[c] && cmin[e] < cmin[c])) ++pos;
    }
    cpos[c] = pos;
  }
  __syncthreads();
  const double kf = floor(__dadd_rn(__dmul_rn(keep_ratio, double(G)), 0.5));
  const int K = kf < 1.0 ? 1 : (kf > double(G) ? G : int(kf));
  for (int i = lane; i < G; i += 64) {
    const int ti = mdap[i] ? 0 : 1;
    int ri = 0;
    for (int j = 0; j < G; ++j)
      ri += (cls[j] == cls[i] && (mdap[j] ? 0 : 1) == ti && vpos[j] < vpos[i]);
    rank[i] = ri;
  }
  __syncthreads();
  for (int i = lane; i < G; i += 64) {
    // key(i) = (tier, rank within class tier, class position); keep the K smallest
    const int ti = mdap[i] ? 0 : 1, ri = rank[i], pi = cpos[cls[i]];
    int smaller = 0;
    for (int j = 0; j < G; ++j) {
      const int tj = mdap[j] ? 0 : 1, rj = rank[j], pj = cpos[cls[j]];
      smaller += (tj != ti) ? (tj < ti) : (rj != ri ? rj < ri : pj < pi);
    }
    keep_mask[g0 + i] = smaller < K ? 1 : 0;
  }
}

// ---------------------------------------------------------------------------- K3b
// DP alignment (Alg. 1 after the union of the per-question sets): while the kept count is
// not a multiple of d, add the unselected trajectory with the highest |A|, round-robin over
// the questions.  One block: count the kept set; rank every unselected member of a valid
// question by (|A| descending, index); one thread deals the rounds to get t_q, the number of
// members question q contributes; members of rank < t_q are kept.
__global__ __launch_bounds__(1024) void dp_fill_kernel(
    uint8_t* __restrict__ keep_mask, const float* __restrict__ adv,
    const int32_t* __restrict__ group_off, const uint8_t* __restrict__ group_valid, int32_t Q,
    int32_t N, int32_t max_group, int32_t d, int32_t* __restrict__ frank,
    int32_t* __restrict__ unsel, int32_t* __restrict__ take, int32_t* __restrict__ status) {
  __shared__ int32_t red[16];
  __shared__ int32_t need_s;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int c = 0;
  for (int i = tid; i < N; i += blockDim.x) c += keep_mask[i] ? 1 : 0;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o, 64);
  if (lane == 0) red[wv] = c;
  __syncthreads();
  if (tid == 0) {
    int kept = 0;
    for (int w = 0; w < int(blockDim.x >> 6); ++w) kept += red[w];
    need_s = (d - kept % d) % d;
  }
  __syncthreads();
  if (need_s == 0) return;
  for (int q = tid; q < Q; q += blockDim.x) {
    const int g0 = group_off[q], g1 = group_off[q + 1];
    int u = 0;
    const bool ok = g0 >= 0 && g1 >= g0 && g1 <= N && g1 - g0 <= max_group &&
                    (group_valid == nullptr || group_valid[q] != 0);
    if (ok) {
      for (int i = g0; i < g1; ++i) {
        if (keep_mask[i]) continue;
        const float ai = isfinite(adv[i]) ? fabsf(adv[i]) : 0.0f;
        int r = 0;
        for (int j = g0; j < g1; ++j) {
          if (keep_mask[j]) continue;
          const float aj = isfinite(adv[j]) ? fabsf(adv[j]) : 0.0f;
          r += (aj > ai) || (aj == ai && j < i);
        }
        frank[i] = r;
        ++u;
      }
    }
    unsel[q] = u;
    take[q] = 0;
  }
  __syncthreads();
  if (tid == 0) {
    int need = need_s;
    for (int r = 0; need > 0; ++r) {
      bool any = false;
      for (int q = 0; q < Q && need > 0; ++q) {
        if (unsel[q] > r) {
          take[q] = r + 1;
          --need;
          any = true;
        }
      }
      if (!any) break;
    }
    if (need > 0) set_status(status, FASTRL_SB_FILL_SHORT);
  }
  __syncthreads();
  for (int q = tid; q < Q; q += blockDim.x) {
    const int t = take[q];
    if (t == 0) continue;
    const int g0 = group_off[q], g1 = group_off[q + 1];
    for (int i = g0; i < g1; ++i)
      if (!keep_mask[i] && frank[i] < t) keep_mask[i] = 1;  // ranks were taken above
  }
}

// ---------------------------------------------------------------------------- K4
__global__ __launch_bounds__(1024) void compact_scan_kernel(
    const uint8_t* __restrict__ keep_mask, const int64_t* __restrict__ toff, int32_t N,
    int32_t* __restrict__ kept_traj, int64_t* __restrict__ kept_tok_off,
    int32_t* __restrict__ kpos, int64_t* __restrict__ counts) {
  __shared__ int32_t wc[16];
  __shared__ int64_t wl[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int32_t base_n = 0;
  int64_t base_t = 0;
  for (int c = 0; c < N; c += 1024) {
    const int i = c + tid;
    const int f = (i < N) ? (keep_mask[i] != 0) : 0;
    const int64_t len = f ? (toff[i + 1] - toff[i]) : 0;
    int vn = f;
    int64_t vl = len;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      int tn = __shfl_up(vn, o, 64);
      int64_t tl = __shfl_up(vl, o, 64);
      if (lane >= o) {
        vn += tn;
        vl += tl;
      }
    }
    if (lane == 63) {
      wc[wv] = vn;
      wl[wv] = vl;
    }
    __syncthreads();
    int32_t pn = 0, totn = 0;
    int64_t pl = 0, totl = 0;
    for (int w = 0; w < 16; ++w) {
      if (w < wv) {
        pn += wc[w];
        pl += wl[w];
      }
      totn += wc[w];
      totl += wl[w];
    }
    if (i < N) {
      const int32_t pos = base_n + pn + vn - f;
      kpos[i] = f ? pos : -1;
      if (f) {
        kept_traj[pos] = i;
        kept_tok_off[pos] = base_t + pl + vl - len;
      }
    }
    base_n += totn;
    base_t += totl;
    __syncthreads();
  }
  if (tid == 0) {
    kept_tok_off[base_n] = base_t;
    counts[0] = base_n;
    counts[1] = base_t;
  }
}

// kpos == NULL: every block takes the exclusive sums over the trajectories before its own itself
// (9 bytes of L2 reads each; up to kSelfScan trajectories that is ~2 us inside this launch, against
// ~5 us for the scan as a launch of its own) and writes its entries of kept_traj and kept_tok_off.
constexpr int kSelfScan = 4096;
__global__ __launch_bounds__(256) void compact_fill_kernel(
    const uint8_t* __restrict__ keep_mask, const int32_t* __restrict__ kpos,
    const int64_t* __restrict__ toff, int32_t N, int32_t* __restrict__ kept_traj,
    int64_t* __restrict__ kept_tok_off, int64_t* __restrict__ counts,
    int32_t* __restrict__ tok_src) {
  const int i = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t a = toff[i], L = toff[i + 1] - a;
  int64_t dst;
  if (kpos) {
    const int pos = kpos[i];
    if (pos < 0) return;
    dst = kept_tok_off[pos];
  } else {
    __shared__ int32_t wc[4];
    __shared__ int64_t wl[4];
    const int kept = keep_mask[i] != 0;
    if (!kept && i != N - 1) return;
    int32_t n = 0;
    int64_t len = 0;
    for (int j = tid; j < i; j += 256) {
      if (keep_mask[j]) {
        ++n;
        len += toff[j + 1] - toff[j];
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      n += __shfl_xor(n, o, 64);
      len += __shfl_xor(len, o, 64);
    }
    if (lane == 0) {
      wc[wv] = n;
      wl[wv] = len;
    }
    __syncthreads();
    n = wc[0] + wc[1] + wc[2] + wc[3];
    dst = wl[0] + wl[1] + wl[2] + wl[3];
    if (tid == 0) {
      if (kept) {
        kept_traj[n] = i;
        kept_tok_off[n] = dst;
      }
      if (i == N - 1) {
        kept_tok_off[n + kept] = dst + (kept ? L : 0);
        counts[0] = n + kept;
        counts[1] = dst + (kept ? L : 0);
      }
    }
    if (!kept) return;
  }
  for (int64_t t = tid; t < L; t += 256) tok_src[dst + t] = int32_t(a + t);
}

// ---------------------------------------------------------------------------- host
size_t prune_workspace(int32_t Q, int32_t N, int64_t T_total, int32_t max_group) {
  Carver c(nullptr);
  c.take<uint64_t>(size_t(T_total > 0 ? T_total : 1));
  c.take<int32_t>(size_t(N + 1));
  c.take<uint64_t>(size_t(N + 1) * ((max_group + 63) / 64));
  c.take<int2>(size_t(N + 1));
  c.take<int32_t>(size_t(N + 1));
  c.take<int32_t>(size_t(N + 1));
  c.take<int32_t>(size_t(N + 1));
  c.take<int32_t>(size_t(Q + 1));
  c.take<int32_t>(size_t(Q + 1));
  return c.size();
}

// K1 and K2 with one kind of set
template <typename S>
static int launch_sets(const int32_t* token_ids, const int64_t* toff, int64_t T_total,
                       const int32_t* group_off, const int32_t* cls, int32_t Q, int32_t N,
                       int32_t max_group, int32_t max_len, int32_t V, int32_t ngram_n,
                       int32_t tau_num, int32_t tau_den, uint64_t* keys, int32_t* nuniq,
                       int2* owner, uint64_t* conflict, int32_t* status, hipStream_t stream) {
  const size_t shm = size_t(S::words(V, max_len)) * 4;
  if (N > 0) {
    if (shm > 64 * 1024)
      FR_HIP(hipFuncSetAttribute((const void*)ngram_set_kernel<S>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(shm)));
    hipLaunchKernelGGL((ngram_set_kernel<S>), dim3(N), dim3(256), shm, stream, token_ids, toff,
                       T_total, V, ngram_n, max_len, keys, nuniq, group_off, Q, N, max_group, owner,
                       status);
    FR_LAUNCHED();
  }
  if (Q > 0 && N > 0) {
    // (the sizes: see pair_conflict_kernel)
    const bool many = N >= 4096 && N <= 64 * int64_t(Q);
    struct {
      decltype(&pair_conflict_kernel<S, 512, 4>) kernel;
      int threads;
    } pair;
    if constexpr (std::is_same<S, BitSet>::value) {
      if (many && max_len <= 512) pair = {pair_conflict_kernel<S, 256, 8>, 256};
      else pair = {pair_conflict_kernel<S, 512, 8>, 512};
    } else if (max_len <= 512) {
      if (many) pair = {pair_conflict_kernel<S, 128, 2>, 128};
      else pair = {pair_conflict_kernel<S, 512, 2>, 512};
    } else {
      if (many && max_len <= 1024) pair = {pair_conflict_kernel<S, 256, 4>, 256};
      else pair = {pair_conflict_kernel<S, 512, 4>, 512};
    }
    if (shm > 64 * 1024)
      FR_HIP(hipFuncSetAttribute((const void*)pair.kernel,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(shm)));
    for (int64_t t0 = 0; t0 < N; t0 += kPairBlocks) {
      const unsigned blocks = unsigned(N - t0 < kPairBlocks ? N - t0 : kPairBlocks);
      hipLaunchKernelGGL(pair.kernel, dim3(blocks), dim3(pair.threads), shm, stream, toff, group_off,
                         cls, keys, nuniq, owner, int32_t(t0), Q, N, V, max_group, tau_num, tau_den,
                         conflict);
      FR_LAUNCHED();
    }
  }
  return FASTRL_OK;
}

int launch_prune(const int32_t* token_ids, const int64_t* toff, int64_t T_total,
                 const float* rewards, const int32_t* group_off, const int32_t* class_id,
                 const float* adv, double group_eps, const uint8_t* group_valid, int32_t Q,
                 int32_t N, int32_t max_group, int32_t max_len, int32_t V, int32_t ngram_n,
                 int32_t tau_num, int32_t tau_den, double keep_ratio, uint8_t* keep_mask,
                 int32_t* mdap_count, int32_t* class_out, int32_t dp_align, int32_t* kept_traj,
                 int64_t* kept_tok_off, int32_t* tok_src, int64_t* counts, int32_t* status,
                 void* ws, hipStream_t stream) {
  Carver c(ws);
  uint64_t* keys = c.take<uint64_t>(size_t(T_total > 0 ? T_total : 1));
  int32_t* nuniq = c.take<int32_t>(size_t(N + 1));
  uint64_t* conflict = c.take<uint64_t>(size_t(N + 1) * ((max_group + 63) / 64));
  int2* owner = c.take<int2>(size_t(N + 1));
  int32_t* kpos = c.take<int32_t>(size_t(N + 1));
  int32_t* cls_eps = c.take<int32_t>(size_t(N + 1));
  int32_t* frank = c.take<int32_t>(size_t(N + 1));
  int32_t* unsel = c.take<int32_t>(size_t(Q + 1));
  int32_t* take = c.take<int32_t>(size_t(Q + 1));
  const int32_t* cls = class_id;
  if (group_eps > 0.0 && Q > 0) {
    hipLaunchKernelGGL(group_eps_kernel, dim3(Q), dim3(64), 0, stream, adv, group_off, N,
                       max_group, group_eps, cls_eps, status);
    FR_LAUNCHED();
    cls = cls_eps;
  }
  const bool bits = ngram_n == 1 && V <= kMaxBitVocab;
  FR_TRY((bits ? launch_sets<BitSet> : launch_sets<HashSet>)(
      token_ids, toff, T_total, group_off, cls, Q, N, max_group, max_len, V, ngram_n, tau_num,
      tau_den, keys, nuniq, owner, conflict, status, stream));
  if (Q > 0) {
    hipLaunchKernelGGL(select_kernel, dim3(Q), dim3(64), 0, stream, rewards, group_off, cls,
                       adv, group_valid, N, max_group, keep_ratio, conflict, owner,
                       keep_mask, mdap_count, class_out, status);
    FR_LAUNCHED();
    if (dp_align > 1) {
      hipLaunchKernelGGL(dp_fill_kernel, dim3(1), dim3(1024), 0, stream, keep_mask, adv,
                         group_off, group_valid, Q, N, max_group, dp_align, frank, unsel, take,
                         status);
      FR_LAUNCHED();
    }
  }
  const bool self_scan = N > 0 && N <= kSelfScan;
  if (!self_scan) {
    hipLaunchKernelGGL(compact_scan_kernel, dim3(1), dim3(1024), 0, stream, keep_mask, toff, N,
                       kept_traj, kept_tok_off, kpos, counts);
    FR_LAUNCHED();
  }
  if (N > 0) {
    hipLaunchKernelGGL(compact_fill_kernel, dim3(N), dim3(256), 0, stream, keep_mask,
                       self_scan ? (const int32_t*)nullptr : kpos, toff, N, kept_traj,
                       kept_tok_off, counts, tok_src);
    FR_LAUNCHED();
  }
  return FASTRL_OK;
}

}  // namespace fastrl
