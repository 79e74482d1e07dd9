// List plan (paper, Section 4.1, with a tile of kListWaves * DW documents; the
// arrays are laid out in common.h): per tile the sorted feature union, and per
// (stage of kListRows union rows, wave) the list of its documents' memberships
// that search_list.h walks.
//
// One workgroup of kListWaves waves per tile.  The features' counts in LDS
// (dense form) give the dense rows and the rest of the union as bitmaps; with a
// prefix count per word, a feature's union row is one LDS read and a bit count.  Wave w
// reads its DW documents' features three times (they stay in the L2): to mark or
// count them, to count its lists' lengths (and set its documents' dense-row
// masks), and to place the entries; a document's features ascend, so those of
// one stage are a run of neighbouring lanes whose first lane owns the counter.
// Only wave w touches list (stage, w), in document order, so the plan is the
// same on every run.  Bound: the latency of the document reads (perm, indptr,
// then indices), which four documents in flight per wave and several workgroups
// per CU hide.
#include "common.h"

namespace som {
namespace {

constexpr int kThreads = kListWaves * 64;
constexpr int S = kListWaves, R = kListRows;

// Slot row of union row k of a stage: the search loads rows 4 * half + i of each
// wave's eight as its i-th pair.
__device__ __forceinline__ uint32_t slot_row(uint32_t k) { return (k & ~7u) | ((k & 3u) << 1) | ((k >> 2) & 1u); }

// Stage capacities of each tile and, with `super` given, the nonzeros of its
// 64-document super-tiles rounded up to kernel 3's 16-entry stages (the offsets
// that kernel's phases are taken from).  One wave per tile.
__global__ void __launch_bounds__(256)
k_list_nnz(const int32_t* __restrict__ indptr, const int32_t* __restrict__ perm, int64_t B, int D, int64_t ntiles,
           int32_t* __restrict__ tile_caps, int32_t* __restrict__ super) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (t >= ntiles) return;
  const int lane = threadIdx.x & 63;
  int32_t s = 0;
  for (int k = lane; k < D; k += 64) {
    const int64_t p = t * D + k;
    int32_t n = 0;
    if (p < B) {
      const int64_t d = perm ? static_cast<int64_t>(perm[p]) : p;
      n = indptr[d + 1] - indptr[d];
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) n += __shfl_xor(n, off, 64);
    if (super && lane == 0 && p < B) super[p / kListSuper] = (n + 15) / 16 * 16;
    s += n;
  }
  if (lane == 0) tile_caps[t] = static_cast<int32_t>((static_cast<int64_t>(s) + R - 1) / R);
}

// Exclusive scan of n values into out[0..n] (out[n] = total; out may be in), one
// workgroup of 1024 threads: 1024 values per step, so the loads stay coalesced.
__device__ void list_scan(const int32_t* in, int64_t n, int32_t* out, int32_t* wsum) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int32_t carry = 0;
  for (int64_t i0 = 0; i0 < n; i0 += 1024) {
    const int64_t i = i0 + tid;
    const int32_t v = i < n ? in[i] : 0;
    int32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int32_t y = __shfl_up(x, off, 64);
      x += lane >= off ? y : 0;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    int32_t before = carry, total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      const int32_t y = wsum[w];
      before += w < wave ? y : 0;
      total += y;
    }
    if (i < n) out[i] = before + x - v;
    carry += total;
    __syncthreads();
  }
  if (tid == 0) out[n] = carry;
}

__global__ void __launch_bounds__(1024)
k_list_scan(const int32_t* caps, int64_t n, int32_t* tile_offset, int32_t* super, int64_t nsuper) {
  __shared__ int32_t wsum[16];
  list_scan(caps, n, tile_offset, wsum);
  if (threadIdx.x == 0) tile_offset[0] = static_cast<int32_t>(kListTag);   // 0, and the plan's mark
  if (super) list_scan(super, nsuper, super, wsum);
}

// Exclusive scan of one value per thread over the workgroup.
__device__ __forceinline__ int32_t block_scan(int32_t v, int32_t* wsum, int32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int32_t x = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t y = __shfl_up(x, off, 64);
    x += lane >= off ? y : 0;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  int32_t before = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < kListWaves; ++w) {
    const int32_t y = wsum[w];
    before += w < wave ? y : 0;
    sum += y;
  }
  __syncthreads();
  *total = sum;
  return before + x - v;
}

// Calls fn(feature, active lane, document of the wave) over the wave's
// documents in order, a document's features in ascending order, 64 at a time;
// every lane of the wave takes part in each call.
template <int DW, typename Fn>
__device__ __forceinline__ void for_each_feature(const int32_t* __restrict__ indices, int32_t begin, int32_t end,
                                                 int lane, Fn fn) {
#pragma unroll 1
  for (int s0 = 0; s0 < DW; s0 += 4) {
    int32_t b[4], e[4], f[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      b[k] = __builtin_amdgcn_readlane(begin, s0 + k);
      e[k] = __builtin_amdgcn_readlane(end, s0 + k);
      f[k] = b[k] + lane < e[k] ? indices[b[k] + lane] : 0;
    }
    int32_t g[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) g[k] = b[k] + 64 + lane < e[k] ? indices[b[k] + 64 + lane] : 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (b[k] < e[k]) fn(f[k], b[k] + lane < e[k], s0 + k);
      if (b[k] + 64 < e[k]) fn(g[k], b[k] + 64 + lane < e[k], s0 + k);
      for (int32_t i = b[k] + 128; i < e[k]; i += 64) fn(i + lane < e[k] ? indices[i + lane] : 0, i + lane < e[k], s0 + k);
    }
  }
}

// The feature at which kernel 3 starts the sweep of super-tile g of ns (see
// search_st.h; the same integers): row s0 * 16 of the super-tile's union, whose
// features are set in `bits`.  A wave's lanes share the work; every lane returns
// it (0 for an empty union).
__device__ int32_t super_start(const uint32_t* bits, int32_t words, const int32_t* __restrict__ super, int64_t g,
                               int64_t ns, int32_t phase_wgs, int lane) {
  const int per = (words + 63) / 64;
  const int w0 = lane * per, w1 = w0 + per < words ? w0 + per : words;
  int32_t c = 0;
  for (int i = w0; i < w1; ++i) c += __popc(bits[i]);
  int32_t x = c;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t y = __shfl_up(x, off, 64);
    x += lane >= off ? y : 0;
  }
  const int32_t cnt = __shfl(x, 63, 64);
  const int32_t nstages = (cnt + 15) / 16;
  int32_t row = 0;
  if (nstages > 1) {
    const int64_t per_xcd = (ns + 7) / 8;
    const int64_t first = g / per_xcd * per_xcd;
    const int64_t end = first + per_xcd < ns ? first + per_xcd : ns;
    const uint64_t o_first = static_cast<uint32_t>(super[first]);
    const uint64_t work = static_cast<uint32_t>(super[end]) - o_first;   // >= cnt > 0
    const uint64_t den = static_cast<uint64_t>(phase_wgs) * work;
    const uint64_t num = (static_cast<uint32_t>(super[g]) - o_first) * static_cast<uint64_t>(end - first) % den;
    row = static_cast<int32_t>(((num << 20) / den * static_cast<uint64_t>(nstages)) >> 20) * 16;
  }
  // the lane whose words hold that row, and the feature
  int32_t f = 0;
  const bool mine = row >= x - c && row < x;
  if (mine) {
    int32_t at = x - c;
    for (int i = w0; i < w1; ++i) {
      const int32_t n = __popc(bits[i]);
      if (row < at + n) {
        uint32_t m = bits[i];
        for (; at < row; ++at) m &= m - 1;
        f = i * 32 + __builtin_ctz(m);
        break;
      }
      at += n;
    }
  }
  const uint64_t who = __ballot(mine);
  return who ? __shfl(f, __builtin_ctzll(who), 64) : 0;
}

// kListDense: find the tile's dense rows (F at most kListDenseMaxF).
// kListSuperOrder: lists in the order kernel 3 sums (DW = 32).
template <int DW, int FORM>
__global__ void __launch_bounds__(kThreads)
k_list_plan(const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices, const int32_t* __restrict__ perm,
            int64_t B, int32_t words, const int32_t* __restrict__ tile_offset, int32_t* __restrict__ tile_count,
            unsigned char* __restrict__ data, uint32_t* __restrict__ start, const int32_t* __restrict__ super,
            int64_t nsuper, int32_t phase_wgs) {
  constexpr bool DENSE = FORM == kListDense, SUPER = FORM == kListSuperOrder;
  constexpr int kSupers = S * DW / kListSuper;   // super-tiles of a tile
  static_assert(!SUPER || kListSuper == 2 * DW, "two waves per super-tile");
  extern __shared__ uint32_t lds[];
  uint32_t* bits = lds;                       // [words] the union's rows with entry lists
  uint32_t* before = lds + words;             // [words] such rows in earlier words
  uint32_t* dense = lds + 2 * words;          // DENSE: [words] the dense rows
  uint32_t* dense_before = lds + 3 * words;   // DENSE: [words]
  uint32_t* mask = lds + 4 * words;           // DENSE: [S * DW][2] the documents' dense rows
  // [visits * S] lengths of the lists, then cursors; before that 16-bit counts of
  // the documents that hold each feature (DENSE), or the super-tiles' unions
  // (SUPER: [kSupers][words])
  uint32_t* counts = DENSE ? mask + 2 * S * DW : lds + 2 * words;
  volatile int32_t* list = reinterpret_cast<volatile int32_t*>(counts);
  __shared__ int32_t wsum[kListWaves];
  __shared__ int32_t starts[kSupers > 0 ? kSupers : 1];   // SUPER: the super-tiles' first features, -1 if empty
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t t = blockIdx.x;
  const int64_t cap0 = static_cast<int64_t>(static_cast<uint32_t>(tile_offset[t]) & ~kListTag);
  unsigned char* base = data + cap0 * list_cap_bytes(SUPER);
  int32_t begin = 0, end = 0;
  {
    const int64_t p = t * (S * DW) + wave * DW + lane;
    if (lane < DW && p < B) {
      const int64_t d = perm ? static_cast<int64_t>(perm[p]) : p;
      begin = indptr[d];
      end = indptr[d + 1];
    }
  }
  // a contiguous run of words per thread
  const int per = (words + kThreads - 1) / kThreads;
  const int w0 = tid * per, w1 = w0 + per < words ? w0 + per : words;
  int32_t nd = 0;   // dense rows
  if (DENSE) {
    for (int i = tid; i < 2 * S * DW; i += kThreads) mask[i] = 0u;
    for (int i = tid; i < words * 16; i += kThreads) counts[i] = 0u;
    __syncthreads();
    for_each_feature<DW>(indices, begin, end, lane, [&](int32_t f, bool on, int) {
      if (on) atomicAdd(&counts[f >> 1], 1u << ((f & 1) * 16));
    });
    __syncthreads();
    int32_t c = 0;
    for (int i = w0; i < w1; ++i) {
      uint32_t any = 0u, many = 0u;
      for (int k = 0; k < 16; ++k) {
        const uint32_t v = counts[i * 16 + k];
        const uint32_t lo = v & 0xffffu, hi = v >> 16;
        any |= (lo ? 1u : 0u) << (2 * k) | (hi ? 1u : 0u) << (2 * k + 1);
        many |= (lo >= S * DW * kListDenseShare / 8 ? 1u : 0u) << (2 * k) |
                (hi >= S * DW * kListDenseShare / 8 ? 1u : 0u) << (2 * k + 1);
      }
      bits[i] = any;
      dense[i] = many;
      c += __popc(many);
    }
    int32_t at = block_scan(c, wsum, &nd);
    // at most one stage of them, the first by id; too few are left to the lists
    nd = nd < kListDenseMin ? 0 : (nd < R ? nd : R);
    for (int i = w0; i < w1; ++i) {
      dense_before[i] = static_cast<uint32_t>(at);
      uint32_t keep = 0u;
      for (uint32_t m = dense[i]; m && at < nd; m &= m - 1, ++at) keep |= m & (~m + 1u);
      dense[i] = keep;
      bits[i] &= ~keep;
    }
  } else if (SUPER) {
    for (int i = tid; i < kSupers * words; i += kThreads) counts[i] = 0u;
    __syncthreads();
    uint32_t* mine = counts + (wave >> 1) * words;
    for_each_feature<DW>(indices, begin, end, lane, [&](int32_t f, bool on, int) {
      if (on) atomicOr(&mine[f >> 5], 1u << (f & 31));
    });
    __syncthreads();
    for (int i = tid; i < words; i += kThreads) {
      uint32_t any = 0u;
#pragma unroll
      for (int k = 0; k < kSupers; ++k) any |= counts[k * words + i];
      bits[i] = any;
    }
    if ((wave & 1) == 0) {
      const int64_t g = t * kSupers + (wave >> 1);
      const int32_t f = g < nsuper ? super_start(mine, words, super, g, nsuper, phase_wgs, lane) : 0;
      const bool some = g < nsuper && super[g + 1] > super[g];
      if (lane == 0) starts[wave >> 1] = some ? f : -1;
    }
  } else {
    for (int i = tid; i < words; i += kThreads) bits[i] = 0u;
    __syncthreads();
    for_each_feature<DW>(indices, begin, end, lane, [&](int32_t f, bool on, int) {
      if (on) atomicOr(&bits[f >> 5], 1u << (f & 31));
    });
  }
  __syncthreads();
  // prefix counts, and the ids: the dense rows, then the others
  int32_t c = 0;
  for (int i = w0; i < w1; ++i) c += __popc(bits[i]);
  int32_t cnt;
  int32_t u = block_scan(c, wsum, &cnt) + nd;
  cnt += nd;
  const int32_t nst = (cnt + R - 1) / R;
  int32_t* ids = reinterpret_cast<int32_t*>(base + (nd ? S * DW * 8 : 0));
  for (int i = w0; i < w1; ++i) {
    before[i] = static_cast<uint32_t>(u);
    for (uint32_t m = bits[i]; m; m &= m - 1) ids[u++] = i * 32 + __builtin_ctz(m);
    if (DENSE) {
      int32_t k = static_cast<int32_t>(dense_before[i]);
      for (uint32_t m = dense[i]; m; m &= m - 1) ids[k++] = i * 32 + __builtin_ctz(m);
    }
  }
  for (int i = cnt + tid; i < nst * R; i += kThreads) ids[i] = 0;
  // SUPER: the sweep starts at the stage q0 of one of the super-tiles' first rows,
  // the one from which the others' first rows come soonest, and goes on past its
  // whole turn to the last of them: nv visits of stages.  This wave's documents
  // take their rows from row_first, visit v_first, on; what lies before it in
  // their order's end is added on the second visit.
  int32_t q0 = 0, nv = nst, row_first = 0, v_first = 0;
  if (SUPER) {
    __syncthreads();   // the prefix counts
    int32_t rows[kSupers > 0 ? kSupers : 1];
#pragma unroll
    for (int k = 0; k < kSupers; ++k) {
      const int32_t f = starts[k];
      rows[k] = f < 0 ? -1 : static_cast<int32_t>(before[f >> 5]) + __popc(bits[f >> 5] & ((1u << (f & 31)) - 1u));
    }
    int32_t most = nst + 1;
#pragma unroll
    for (int i = 0; i < kSupers; ++i) {
      if (rows[i] < 0) continue;
      int32_t far = 0;
#pragma unroll
      for (int k = 0; k < kSupers; ++k) {
        if (rows[k] < 0) continue;
        const int32_t v = rows[k] / R - rows[i] / R;
        const int32_t e = (v < 0 ? v + nst : v) + (rows[k] % R ? 1 : 0);
        far = e > far ? e : far;
      }
      if (far < most) {
        most = far;
        q0 = rows[i] / R;
        nv = nst + far;
      }
    }
    row_first = rows[0];
#pragma unroll
    for (int k = 1; k < kSupers; ++k) row_first = (wave >> 1) == k ? rows[k] : row_first;
    v_first = row_first / R - q0;
    v_first += v_first < 0 ? nst : 0;
  }
  for (int i = tid; i < nv * S; i += kThreads) list[i] = 0;   // (the counts are done with)
  if (tid == 0)
    tile_count[t] = SUPER ? static_cast<int32_t>(static_cast<uint32_t>(nst | q0 << 11) |
                                                 static_cast<uint32_t>(nv - nst) << 21)
                          : nst | nd << 16;
  __syncthreads();

  // A call's lanes by visit of a stage: the first lane of each run (leader), the
  // entries of the run, and each lane's place among them.  A dense row's lane
  // counts with the row that would stand in its place.
  struct Run {
    int32_t row, list, entries, place;
    bool leader, entry;
  };
  auto run_of = [&](int32_t f, bool on) {
    Run r;
    const uint32_t m = 1u << (f & 31), w = bits[f >> 5];
    r.row = static_cast<int32_t>(before[f >> 5]) + __popc(w & (m - 1u));
    r.entry = on && (w & m) != 0u;
    int32_t visit = on ? (r.row / R < nst ? r.row / R : nst - 1) : -1;
    if (SUPER && on) {
      visit -= q0;
      visit += visit < 0 ? nst : 0;
      if (visit < v_first || (visit == v_first && r.row < row_first)) visit += nst;
    }
    r.list = visit * S + wave;
    const int32_t prev = __shfl_up(visit, 1, 64);
    r.leader = on && (lane == 0 || prev != visit);
    const uint64_t leaders = __ballot(r.leader), with = __ballot(r.entry);
    const uint64_t below = (1ull << lane) - 1ull, upto = (below << 1) | 1ull;
    const uint64_t later = leaders & ~upto;
    const uint64_t until = later ? (later & (~later + 1ull)) - 1ull : ~0ull;    // lanes before the next leader
    const int first = 63 - __builtin_clzll((leaders & upto) | 1ull);
    const uint64_t run = with & until & ~((1ull << first) - 1ull);
    r.entries = __popcll(run);
    r.place = __popcll(run & below);
    return r;
  };
  for_each_feature<DW>(indices, begin, end, lane, [&](int32_t f, bool on, int s) {
    const Run r = run_of(f, on);
    if (r.leader) list[r.list] += r.entries;
    if (DENSE && on && !r.entry) {
      const uint32_t d = slot_row(dense_before[f >> 5] + __popc(dense[f >> 5] & ((1u << (f & 31)) - 1u)));
      atomicOr(&mask[2 * (wave * DW + s) + (d >> 5)], 1u << (d & 31));
    }
  });
  __syncthreads();
  if (nd)
    for (int i = tid; i < 2 * S * DW; i += kThreads) reinterpret_cast<uint32_t*>(base)[i] = mask[i];
  // starts of the lists in units of four entries; lengths become cursors
  uint32_t* st = start + cap0 * list_cap_lists(SUPER) + t;
  int32_t units = 0;
  for (int i0 = 0; i0 < nv * S; i0 += kThreads) {
    const int i = i0 + tid;
    const int32_t v = i < nv * S ? (list[i] + 3) / 4 : 0;
    int32_t sum;
    const int32_t at = units + block_scan(v, wsum, &sum);
    if (i < nv * S) {
      st[i] = static_cast<uint32_t>(at);
      list[i] = at * 4;
    }
    units += sum;
  }
  if (tid == 0) st[nv * S] = static_cast<uint32_t>(units);
  __syncthreads();
  uint16_t* entries = reinterpret_cast<uint16_t*>(ids + nst * R);
  for_each_feature<DW>(indices, begin, end, lane, [&](int32_t f, bool on, int s) {
    const Run r = run_of(f, on);
    if (r.entry) {
      entries[list[r.list] + r.place] = static_cast<uint16_t>(slot_row(r.row % R) * kListRowBytes + s);
    }
    __builtin_amdgcn_wave_barrier();
    if (r.leader) list[r.list] += r.entries;   // after every lane's read: LDS operations of a wave keep their order
    __builtin_amdgcn_wave_barrier();
  });
  __syncthreads();
  for (int i = tid; i < nv * S; i += kThreads)
    for (int32_t k = list[i]; k & 3; ++k) entries[k] = static_cast<uint16_t>(DW);   // slot row 0 into the spare register
}

// LDS of k_list_plan: tables, then lists in the space of what precedes them.
size_t plan_lds_bytes(int form, size_t D, size_t words, size_t stages) {
  const size_t lists = (form == kListSuperOrder ? 2 : 1) * stages * S;
  const size_t first = form == kListDense ? 16 * words : form == kListSuperOrder ? 4 * words : 0;
  return sizeof(uint32_t) * ((form == kListDense ? 4 * words + 2 * D : 2 * words) + (lists > first ? lists : first));
}

}  // namespace

hipError_t launch_list_plan(const int32_t* indptr, const int32_t* indices, int64_t B, int64_t F,
                            const int32_t* perm, int DW, int form, int32_t* tile_offset, int32_t* tile_count,
                            unsigned char* data, uint32_t* start, int32_t* super, hipStream_t stream) {
  if (F > kListMaxF || (DW != 16 && DW != 32) || (form == kListSuperOrder && DW != 32)) return hipErrorInvalidValue;
  const int D = S * DW;
  const int64_t ntiles = (B + D - 1) / D;
  if (form == kListDense && (DW != 32 || F > kListDenseMaxF)) form = kListPlain;
  const int64_t nsuper = form == kListSuperOrder ? (B + kListSuper - 1) / kListSuper : 0;
  int32_t phase_wgs = 0;
  if (nsuper) {
    const hipError_t e = st_phase_wgs(8, kListSuper / 8, &phase_wgs);   // kernel 3's automatic super-tile
    if (e != hipSuccess) return e;
  } else {
    super = nullptr;
  }
  hipLaunchKernelGGL(k_list_nnz, dim3(static_cast<uint32_t>((ntiles + 3) / 4)), dim3(256), 0, stream, indptr, perm, B,
                     D, ntiles, tile_count, super);
  hipLaunchKernelGGL(k_list_scan, dim3(1), dim3(1024), 0, stream, tile_count, ntiles, tile_offset, super, nsuper);
  const int32_t words = static_cast<int32_t>((F + 31) / 32);
  const size_t stages = static_cast<size_t>((F + R - 1) / R);
  const size_t bytes = plan_lds_bytes(form, D, words, stages);
  auto* kernel = DW == 16                ? &k_list_plan<16, kListPlain>
                 : form == kListDense      ? &k_list_plan<32, kListDense>
                 : form == kListSuperOrder ? &k_list_plan<32, kListSuperOrder>
                                           : &k_list_plan<32, kListPlain>;
  const size_t most = plan_lds_bytes(form, D, form == kListDense ? kListDenseMaxF / 32 : kListMaxF / 32,
                                     form == kListDense ? kListDenseMaxF / R : kListMaxF / R);
  const hipError_t e = allow_lds(kernel, most);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(static_cast<uint32_t>(ntiles)), dim3(kThreads), bytes, stream, indptr, indices, perm,
                     B, words, tile_offset, tile_count, data, start, super, nsuper, phase_wgs);
  return hipGetLastError();
}

}  // namespace som
