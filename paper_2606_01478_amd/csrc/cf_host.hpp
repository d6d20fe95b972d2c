// Host-only part of the runtime behind include/cfsim.h: everything that needs
// no device -- descriptor validation, the derived per-world records, the
// per-world tile lists of uneven batches, the autotune cache file, and the
// checkpoint tag that ties a backward call to the forward that filled its
// checkpoint buffer. Plain C++17 (no HIP): the library links it, and a CPU
// test builds it on its own under AddressSanitizer and UBSan.
#pragma once
#include <cstdint>
#include <initializer_list>
#include <map>
#include <string>
#include <vector>

#include "../../include/cfsim.h"

namespace cfh {

// ---- descriptor and parameter records -------------------------------------------

// Validates *d; on success fills the per-world drone counts, models and gain
// indices and the total drone count. Returns CF_EINVAL on any violation of the
// cf_desc contract (header), CF_OK otherwise.
cf_status validate_desc(const cf_desc* d, std::vector<int32_t>& counts, std::vector<uint8_t>& models,
                        std::vector<int32_t>& gidx, int64_t* D_out);

// out[0..NREC): the public record r[0..CF_NPARAM) followed by the constants the
// kernels read instead of forming them (reciprocals, inertia differences, the
// reference-speed terms of the first-principles model, c_f / m and the hover
// thrust of the identified model).
void derive_record(const float* r, float* out);

// out[D_STEP..NREC): the coefficients of an RK4 step of length dt of a world of
// `model`, from the record out[0..D_STEP) that derive_record formed.
void derive_step(int model, float dt, float* out);

// True when the rotor drag-torque polynomial is the thrust polynomial times one
// constant kappa (t_j = kappa k_j for j = 0, 1, 2, to 2^-20 relative); *kappa
// receives it. The reduced kernel variants then form the yaw torque from the
// thrust differences (coefficients kappa * yaw mixing, D_TZK).
bool torque_proportional(const float* r, double* kappa);

// ---- uneven batches --------------------------------------------------------------

struct Tile {
    int world, first, count, model;
};

// Per-world tiles of at most `tile` drones {world, first drone, count, model}:
// first-principles tiles first, within a model in longest-processing-time
// order (cost = 64-lane waves x model cost, ties by position). *n_fp receives
// the number of first-principles tiles.
std::vector<Tile> tile_list(const std::vector<int32_t>& counts, const std::vector<int64_t>& offsets,
                            const std::vector<uint8_t>& models, int control, int tile, int* n_fp);

// Packed tiles of the held-step kernels: the drones of each model listed world
// after world (first-principles worlds first, worlds in index order, a world's
// drones in order) in *list, cut into tiles of `tile` consecutive entries
// {first entry, count, model}, so that every tile but each model's last is full
// and a tile may span several worlds of its model. *n_fp receives the number of
// first-principles tiles (they come first).
struct PackedTile {
    int first, count, model;
};
std::vector<PackedTile> packed_tiles(const std::vector<int32_t>& counts, const std::vector<int64_t>& offsets,
                                     const std::vector<uint8_t>& models, int tile, std::vector<int32_t>* list,
                                     int* n_fp);

// ---- sums over the drones (gain and policy gradients) -----------------------------

// The sums are taken over chunks of consecutive drones, one workgroup each, and then
// over the chunks. 16384 drones give each of a workgroup's 1024 threads 16; beyond
// 1024 chunks (2^24 drones) the chunk grows instead of their number, so that the
// partial sums stay bounded. The launch and its scratch both follow from these.
constexpr int64_t SUM_CHUNK = 16384;
constexpr int SUM_MAX_CHUNKS = 1024;
// drones per chunk: a multiple of the 4096 that a workgroup reads at a time
int64_t sum_chunk(int64_t D);
int sum_chunks(int64_t D);
// floats of the partial sums of nc components per gain
size_t sum_part_floats(int n_gains, int nc, int64_t D);

// ---- scratch of a rollout's backward -----------------------------------------------

// What of a backward call decides its scratch: reward: the reward objective; eight: a
// figure-eight objective; hidden: width of its policies (0: linear feedback or none);
// gains: 0 when no gain gradient is asked for.
struct BackwardShape {
    int T, K, S;
    int64_t D;
    bool reward, eight;
    int hidden, gains;
};
// Floats of the static scratch that cf_rollout_backward_noalloc asks for (the sum that its
// contract states, each term rounded up to 64). The layouts that the kernels of a batch
// use take no more, so what is refused does not depend on them.
size_t noalloc_floats(const BackwardShape& b);
// workgroups of the sum over a policy's records
int policy_blocks(int64_t records);

// Tries the sizes in order (most wanted first) with grow(size), a status of which
// `too_large` moves on to the next size and any other ends the search. *got receives the
// index of the last size tried; returns its status.
template <class Status, class Grow>
Status grow_to_any(std::initializer_list<size_t> sizes, Status too_large, size_t* got, Grow&& grow) {
    Status s = too_large;
    *got = 0;
    for (size_t n : sizes) {
        s = grow(n);
        if (s != too_large || *got + 1 == sizes.size()) break;
        ++*got;
    }
    return s;
}

// ---- autotune cache ---------------------------------------------------------------

struct LaunchChoice {
    int wq = 0, tile = 64, chunk = 0, split = 1;
    float ms = 0.f;
};

// One line per handle signature: "<key> <wq> <tile> <chunk> <split> <ms>".
// Lookup keeps the last well-formed line of the key; malformed lines are
// skipped. Store rewrites the file with the key's line replaced.
bool cache_lookup(const std::string& path, const std::string& key, LaunchChoice* c);
bool cache_store(const std::string& path, const std::string& key, const LaunchChoice& c);

// ---- checkpoint buffers and their tag ---------------------------------------------

constexpr uint32_t TAG_MAGIC = 0x4b434643u;  // "CFCK"

struct CkptTag {
    uint32_t w[CF_CKPT_TAG_FLOATS];
};

// Floats of a checkpoint buffer for (T, K): ceil(T/K) states [S][D], then for
// the reward objective the applied commands [T][4][D], then the tag.
int64_t ckpt_floats(int T, int K, int S, int64_t D, int kind);
// Offset (floats) of the applied commands and of the tag inside that buffer.
int64_t ckpt_ubuf_offset(int T, int K, int S, int64_t D);
int64_t ckpt_tag_offset(int T, int K, int S, int64_t D, int kind);

// FNV-1a hash of what of the objective the backward must share with the
// forward: no objective / its kind, which optional inputs are present (gain,
// table, offsets) and its scalar weights.
uint32_t objective_hash(const cf_objective* obj);

// {magic, handle id, generation, T, K, S, D, kind, objective hash, 0.., checksum}
CkptTag make_tag(uint32_t handle_id, uint32_t generation, int T, int K, int S, int64_t D,
                 const cf_objective* obj);
bool tag_well_formed(const CkptTag& t);

// The tags of the forwards with a checkpoint buffer run on one handle, by
// buffer address (bounded; the oldest generation is dropped first). A backward
// is accepted only for a buffer whose latest forward on this handle had the
// same T, K, state size, drone count and objective; the tag returned is what
// the device then finds in the buffer unless it was overwritten since.
class CkptRegistry {
public:
    explicit CkptRegistry(size_t capacity = 256) : cap_(capacity) {}
    void record(const void* ckpt, const CkptTag& tag);
    cf_status match(const void* ckpt, int T, int K, int S, int64_t D, const cf_objective* obj,
                    CkptTag* out) const;
    size_t size() const { return map_.size(); }

private:
    size_t cap_;
    std::map<const void*, CkptTag> map_;
};

}  // namespace cfh
