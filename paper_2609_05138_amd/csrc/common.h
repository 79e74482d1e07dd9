// Internal declarations shared by the HIP translation units of libsom.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace som {

// Packed argmin key: the high 32 bits are the distance mapped to an unsigned
// integer whose order matches the float order, the low 32 bits the neuron
// index.  The unsigned 64-bit minimum of two keys is then the smaller
// distance, and on equal distances the lower index -- associative and
// commutative, so the reduction order never changes the answer.
__device__ __forceinline__ uint32_t ordered_bits(float d) {
  uint32_t u = __float_as_uint(d);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float from_ordered_bits(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

__device__ __forceinline__ uint64_t pack_key(float d, uint32_t j) {
  return (static_cast<uint64_t>(ordered_bits(d)) << 32) | j;
}

constexpr uint64_t kNoKey = ~0ull;

// Lets `kernel` be launched with up to `most` bytes of dynamic LDS.  `most` is the
// most that any call asks for: the limit belongs to the process, and a call that
// set it to its own need would lower it under another thread's launch.
template <typename F>
hipError_t allow_lds(F* kernel, size_t most) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             static_cast<int>(most));
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ---------------------------------------------------------------------------
// Launchers (each enqueues on `stream` and returns the launch status).
// ---------------------------------------------------------------------------

// Codebook storage types (SearchArgs::weights, launch_norms).
constexpr int kWeightsF32 = 0;
constexpr int kWeightsF16 = 1;

hipError_t launch_norms(const void* W, int weights, int64_t F, int64_t N, int64_t ldw, float* norms,
                        hipStream_t stream);

// CSR (and optional permutation) checks; sets *flag (device int) nonzero on failure.
hipError_t launch_validate(const int32_t* indptr, const int32_t* indices, int64_t B, int64_t F,
                           int64_t nnz, const int32_t* perm, int32_t* seen, int32_t* flag,
                           hipStream_t stream);

// Tile plan: tile_offset[ntiles+1] (exclusive scan of per-tile nonzeros),
// tile_count[ntiles], union_feat / union_mask (see som_tile_plan).  With
// stage_masks (tiles of 64, 128 or 256 documents: the shared-union search's
// document-major form) each tile's region is rounded up to whole 16-entry
// stages and each stage's masks are stored document-major: 16-bit word s of
// the stage (at the stage's first mask word) holds bit r set iff document s
// holds entry r of the stage.
hipError_t launch_tile_plan(const int32_t* indptr, const int32_t* indices, int64_t B, int64_t F,
                            const int32_t* perm, int T, int32_t* tile_offset, int32_t* tile_count,
                            int32_t* union_feat, uint32_t* union_mask, hipStream_t stream,
                            bool stage_masks = false);

// List plan (for the list form of the shared-union search, search_list.h), in
// tiles of kListWaves * DW documents: a tile's feature union in ascending order,
// cut into stages of kListRows, and per (visit of a stage, wave) a list of 16-bit
// entries, one per membership: the document's place in the wave in the low bits,
// the row's slot offset (a multiple of kListRowBytes) above; padded to whole units
// of four.  Three forms, which fix the order the search sums in:
//   kListPlain       one visit per stage, swept in ascending order (or, without
//                    dense rows, from the search's own phase)
//   kListDense       rows that at least 3/8 of a 256-document tile's documents
//                    hold (its dense rows, where there are kListDenseMin of them
//                    or more, at most kListRows) come before the others and have
//                    no entries: each document has a 64-bit mask of those it
//                    holds.  Swept from the search's own phase
//   kListSuperOrder  256-document tiles, summed as kernel 3 sums the four
//                    64-document super-tiles they hold: a document's rows from
//                    its super-tile's first feature (rotated sweep) on, then those
//                    before it.  The sweep starts at a stage q0 and makes nv
//                    visits, wrapping round, at most twice the stages: one turn,
//                    and on to the last super-tile's first row.  `super` (the
//                    exclusive scan of the super-tiles' nonzeros, rounded up to 16)
//                    is scratch of the plan's making
// Space is counted in stage capacities: ceil(nnz / kListRows) per tile
// bound its stages (a union row has a nonzero); tile_offset is their exclusive
// scan, with kListTag set in its first word (a tile plan's, at the same place, is
// 0), so that a search can tell the plans apart; tile_count the stages in use, and above them (bit 16 on) the dense rows,
// or (kListSuperOrder: from bits 11 and 21 on) q0 and nv less the stages.  A
// tile's bytes in `data` start at tile_offset * list_cap_bytes: with dense rows
// its documents' masks (eight bytes each, no more than the dense rows' entries
// would take), the ids of its stages (int32, padded with 0), then its lists.  Its
// words of `start` begin at tile_offset * list_cap_lists + t: the start of list
// i = visit * kListWaves + wave, in units from the tile's first list; list i + 1
// follows.
constexpr int kListWaves = 8;
constexpr int kListRows = 64;
constexpr int kListRowBytes = 512;
constexpr uint32_t kListTag = 0x80000000u;
enum ListForm { kListPlain = 0, kListDense = 1, kListSuperOrder = 2 };
constexpr int kListSuper = 64;       // documents of a kernel-3 super-tile
// per stage: lists, and bytes of ids, entries and the lists' padding
__host__ __device__ constexpr int list_cap_lists(bool super_order) { return kListWaves * (super_order ? 2 : 1); }
__host__ __device__ constexpr int list_cap_bytes(bool super_order) {
  return kListRows * (4 + 2) + list_cap_lists(super_order) * 3 * 2;
}
constexpr int kListStageWork = 128;  // a stage's fixed cost in entries, for the phase of rotated sweeps
constexpr int kListPhaseWgs = 96;    // phase period in workgroups per XCD
constexpr int64_t kListMaxF = 65536;  // the plan kernel's tables fit the LDS
static_assert(kListMaxF / kListRows <= 1024, "a tile's stages fit the fields of its count");
constexpr int kListDenseShare = 3;            // a dense row's holders: eighths of the documents
constexpr int kListDenseMin = 16;
constexpr int64_t kListDenseMaxF = 32768;     // the plan kernel's counts fit the LDS
// masks: kListWaves * DW * 8 bytes; entries saved: kListDenseMin rows of
// kListWaves * DW * kListDenseShare / 8 entries of 2 bytes
static_assert(kListDenseMin * 2 * kListDenseShare >= 8 * 8, "the masks fit the space of the entries they replace");
static_assert(list_cap_bytes(false) % 16 == 0 && list_cap_bytes(true) % 16 == 0,
              "a tile's ids are read 16 bytes at a time");
hipError_t launch_list_plan(const int32_t* indptr, const int32_t* indices, int64_t B, int64_t F,
                            const int32_t* perm, int DW, int form, int32_t* tile_offset, int32_t* tile_count,
                            unsigned char* data, uint32_t* start, int32_t* super, hipStream_t stream);

// Document-group plan (for the documents-on-lanes search): per group of D
// consecutive documents of the tiled order, the sorted feature union and the
// union position of every nonzero.
hipError_t launch_group_plan(const int32_t* indptr, const int32_t* indices, int64_t B, int64_t F,
                             const int32_t* perm, int D, int32_t* group_offset, int32_t* group_count,
                             int32_t* group_feat, int32_t* entry_pos, hipStream_t stream);

// Block index -> (tile or tile-group index, neuron slice) of a kernel-1/3
// launch over a grid of nx (a multiple of 8) x nslices workgroups, dealt to
// the XCDs round-robin in linear order.  XCD x owns the contiguous tile range
// [x * nx/8, (x+1) * nx/8); it visits the neuron slices in chunks of q, and
// inside a chunk its tiles in turn with the chunk's slices back to back (the
// last chunk may hold fewer than q slices).  q = 1 is slice-major order.
__host__ __device__ inline void chunked_block(uint64_t lin, uint64_t nx, uint64_t nslices, uint64_t q,
                                              uint64_t* unit, uint64_t* slice) {
  const uint64_t xcd = lin % 8, j = lin / 8, per = nx / 8;
  const uint64_t full = nslices / q, rest = nslices - full * q;
  const uint64_t chunk = j / (per * q);
  const uint64_t r = chunk < full ? j - chunk * per * q : j - full * per * q;
  const uint64_t qq = chunk < full ? q : rest;
  *unit = xcd * per + r / qq;
  *slice = chunk * q + r % qq;
}

// Phase periods of the rotated sweeps (see search.hip): kernel 3 with
// super-tiles of S waves of T documents, in workgroups per XCD; kernel 1
// with T-document tiles, G per workgroup, in tiles per XCD.
hipError_t st_phase_wgs(int T, int S, int32_t* wgs);
hipError_t k1_phase_tiles(int T, int G, int mask_mode, int32_t* tiles);

struct SearchArgs {
  const void* W;    // fp32 or fp16 [F][ldw] (see `weights`)
  int weights;      // kWeightsF32 or kWeightsF16 (kernel 1 only)
  int64_t F, N, ldw;
  const float* norms;
  const int32_t* indptr;
  const int32_t* perm;
  int64_t B;
  int T;            // documents per tile (kernel 3: per wave)
  int K;            // neurons per lane (4 or 8); a slice is 64 * K neurons
  int group;        // tiles (waves) per workgroup, all on the same slice
                    // (kernel 3: waves per super-tile of group * T documents)
  int mask_mode;    // 0 = branch-free fma by the membership bit, 1 = scalar branches
  int64_t ntiles;
  int64_t nchunks;  // neuron slices = ceil(N / (64 * K))
  int64_t tile_base = 0;  // kernel 1 searches tiles [tile_base, tile_end) of the plan
  int64_t tile_end = 0;
  // kernel 3, round-synchronised launches (round_wgs > 0): one launch per
  // (neuron slice, round); XCD x searches super-tiles x * xcd_span +
  // round_base + [0, round_wgs) of slice slice_base
  int32_t schedule = 0;   // 1 = one launch over every slice, 2 = rounds
  int32_t round_wgs = 0;
  int64_t round_base = 0;
  int64_t xcd_span = 0;
  int64_t slice_base = 0;
  // kernels 1 and 3 (one launch over every slice): neuron slices per schedule
  // chunk; the grid's workgroups walk the chunks in turn, and inside a chunk
  // each XCD's tiles with their chunk slices back to back (1 = slice-major)
  int32_t chunk_slices = 1;
  // kernels 1 and 3 (one launch of one-slice chunks; kernel 3
  // document-major): 1 = rotated sweep; phase_wgs is its phase period, in
  // workgroups (kernel 3) or tiles (kernel 1) per XCD, set by the launch.  List
  // form: 1 = from the launch's own phase, 2 = a kListSuperOrder plan
  int32_t rotate = 0;
  int32_t phase_wgs = 0;
  // 1: the launch ends at once unless the plan is of its kernel's kind (list or
  // tile plan, told apart by kListTag): both kinds are launched, one after the other
  int32_t either = 0;
  float* score = nullptr;  // unfused comparator: distances of tiled-order documents
                           // [tile_base * T, ...) go to score[(p - tile_base * T) * N + j]
  const int32_t* tile_offset;
  const int32_t* tile_count;
  const int32_t* union_feat;
  const uint32_t* union_mask;
  const unsigned char* list_data;   // list form (kernel 4)
  const uint32_t* list_start;
  uint64_t* keys;   // [B] packed (distance, index) minima, tiled order
  uint64_t* keys2;  // [B] second-smallest keys, or nullptr when only the BMU is wanted
  // documents-on-lanes search (kernel 2)
  int kernel;       // 1 = neurons on lanes (tile masks), 2 = documents on lanes (groups),
                    // 3 = shared-union super-tiles (tile plan with group * T / 32 mask words),
                    // 4 = their list form (list plan, T documents per wave)
  int slice;        // kernel 2: neurons per slice (32 or 64)
  const int32_t* group_offset;
  const int32_t* group_count;
  const int32_t* group_feat;
  const int32_t* entry_pos;
  int32_t* bmu;
  float* dist;
  int32_t* bmu2;    // with keys2: second-best unit (-1 if none) and its distance (+inf)
  float* dist2;
};

// Initialises the keys, then runs the fused search (launch_kernel: without them).
hipError_t launch_search(const SearchArgs& a, hipStream_t stream);
hipError_t launch_kernel(const SearchArgs& a, hipStream_t stream);
// Kernels 1 and 3 over an fp16 codebook (their own translation unit).
hipError_t launch_search_k1_f16(const SearchArgs& a, hipStream_t stream);
hipError_t launch_search_st_f16(const SearchArgs& a, hipStream_t stream);
hipError_t launch_search_list_f16(const SearchArgs& a, hipStream_t stream);
// Unfused comparator: kernel 1 writes the distance block of block_docs
// documents at a time into `score`, then a wave-per-row argmin reduces it.
hipError_t launch_unfused(SearchArgs a, int64_t block_docs, hipStream_t stream);
// Decodes the keys into results in input order.
hipError_t launch_merge(const SearchArgs& a, hipStream_t stream);

// Batch-SOM update (update.hip).
constexpr int kUpdateMaxRows = 1024;   // column-blur strip: rows x 32 fp32 in LDS
constexpr int kUpdateMaxCols = 16384;  // row blur: one grid row in LDS
constexpr int kUpdateMaxRadius = 4096;
size_t update_chunk_planes(int64_t F, int64_t N);
hipError_t launch_update_accumulate(const int32_t* indptr, const int32_t* indices, int64_t B, const int32_t* bmu,
                                    int64_t F, int64_t N, uint32_t* acc, int64_t ld_acc, uint32_t* count,
                                    hipStream_t stream);
hipError_t launch_update_finish(void* W, int weights, int64_t F, int64_t ldw, int rows, int cols, double sigma, int R,
                                const uint32_t* acc, int64_t ld_acc, const uint32_t* count, float* taps,
                                float* den_tmp, float* den, float* chunk, int64_t chunk_planes,
                                hipStream_t stream);

// Read-bandwidth probe (probe.hip): `passes` grid-stride reads of buf.
hipError_t launch_read_probe(const void* buf, int64_t bytes, int32_t passes, uint32_t* sink, hipStream_t stream);
hipError_t launch_lds_probe(int32_t iters, uint32_t* sink, int64_t* bytes, hipStream_t stream);

// Clustering: df histogram, signatures and a bitonic sort of n2 =
// cluster_sort_size(B) (a power of two >= B) (key, position) pairs.
int64_t cluster_sort_size(int64_t B);
hipError_t launch_cluster(const int32_t* indptr, const int32_t* indices, int64_t B, int64_t F,
                          int64_t nnz, int32_t* perm, int32_t* df, uint64_t* keys, uint32_t* vals,
                          hipStream_t stream);

}  // namespace som
