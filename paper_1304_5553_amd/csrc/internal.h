// Internals shared by the translation units that implement the C ABI:
// the handle object, launch-geometry defaults and the variant cache.
#pragma once

#include <atomic>
#include <functional>
#include <map>
#include <set>
#include <unordered_map>

#include "common.h"

namespace hipmr {
// The kernels of one call, in the order looked up (the handle keeps them alive).
struct CallKernels {
    const CodeObject* co[4] = {};
    int n = 0;
};
}  // namespace hipmr

struct hipmr_kernel {
    int refs = 1;                 // changed only under the handle cache's lock
    bool cached = false;          // listed in the handle cache under cache_key
    std::string cache_key;
    hipmr::Program prog;
    int default_vec = 4;          // elements per chunk,
    int stream_vec = 4;           // and of the elementwise kernels and plain reductions
    int ew_ipt = 1;               // elementwise chunks per thread
    bool map_calls = false;       // the map calls functions other than the cheapest
    std::mutex mu;
    std::unordered_map<hipmr::KernelSpec, std::shared_ptr<hipmr::CodeObject>, hipmr::KernelSpecHash> variants;
    hipmr::CallKernels last;                         // kernels of the most recent call
    std::map<std::string, hipmr_launch_config> tuned;  // autotuned geometry per operation
    std::set<std::string> families;                  // operations whose kernels are all loaded (load_family)
};

namespace hipmr {

constexpr int kMaxPartials = 8192;           // stage-1 blocks of one reduce
constexpr int kStage2Block = 256;
// reduce workspace layout: [0, 64 KiB) block partials (FP64 or the
// reduction's type); [64 KiB, 96 KiB) the norm's first-pass partials (max
// |map| per block, float), kept apart so the second pass can read them while
// it writes its own; then its scale, and room to spare.  The norm's second pass exchanges its
// partials within its launch in the upper half of the first 64 KiB, which up
// to 1024 blocks' first-pass partials leave free (32 bytes per block); larger
// grids fold in a launch of their own.
constexpr size_t kAmaxOffset = (size_t)kMaxPartials * 8;
constexpr size_t kNormWordsOffset = kAmaxOffset / 2;
constexpr int kNormWordsBlocks = 1024;
constexpr size_t kWorkspaceBytes = kAmaxOffset + (size_t)kMaxPartials * 4 + 256;
static_assert(kNormWordsBlocks * 8 <= kNormWordsOffset &&
              kNormWordsOffset + kNormWordsBlocks * 32 <= kAmaxOffset, "the norm's words overlap");

// Words that blocks of one launch exchange are 64 bits, accessed atomically:
// a workspace that starts off their alignment is used from the next multiple
// of 8 (the reduce workspace's last 256 bytes leave room for that).
inline char* align_words(void* workspace) { return (char*)(((uintptr_t)workspace + 7) & ~(uintptr_t)7); }

// Default geometry (overridable per call through hipmr_launch_config), from
// sweeps on MI355X at n = 2^28: streaming reads reach their best rate with a
// small resident grid (2 blocks of 256 threads per CU, 4 chunks of 16 bytes
// in flight per thread and array); elementwise kernels, which mix reads and
// writes, do best as one pass over a full grid (one chunk per thread).
constexpr int kEwBlock = 256, kEwIpt = 1, kEwBlocksPerCu = 1 << 20;
constexpr int kEwMixedIpt = 2;               // arrays of different element sizes (see default_stream_shape)
constexpr int kEwScalarBlocksPerCu = 32;     // one-element elementwise kernels
constexpr int kRedBlock = 256, kRedIpt = 4, kRedBlocksPerCu = 2;

hipmr_status resolve_cfg(const hipmr_launch_config* c, int block, int ipt, int vec,
                         int blocks_per_cu, LaunchCfg* out);
hipmr_status get_variant(hipmr_kernel* h, const KernelSpec& spec, std::shared_ptr<CodeObject>* out);
hipmr_status variant_function(hipmr_kernel* h, const KernelSpec& spec, void** fn,
                              CallKernels* used);
void set_last_kernels(hipmr_kernel* h, const CallKernels& used);
// Builds (as one program) and loads every kernel that `op` may use on this
// device at any size, the first time it runs there, so that a later capture
// finds them whatever its size.  Nothing is loaded during a capture.
hipmr_status load_family(hipmr_kernel* h, char op, bool vector, bool idx64, const LaunchCfg& cfg,
                         const char* combine, const char* neutral,
                         const std::function<std::vector<KernelSpec>()>& specs);
// runs the jobs on a thread pool; the first failure's status and message
hipmr_status run_concurrently(const std::vector<std::function<hipmr_status()>>& jobs);
// Element offset at which the chunks start, or -1 for the one-element kernels
// (a map or statement that cannot run on chunks, or an array off its element
// alignment): every written array is aligned for VEC-element chunks there, and
// so are all read ones, or cfg->unaligned is set and those that are not are
// loaded at element alignment.  `out` of `out_size` bytes per element (0: none)
// is written besides the arguments.
long long vector_head(const hipmr_kernel* h, void* const* args, LaunchCfg* cfg,
                      const void* out = nullptr, int out_size = 0);
hipmr_status check_args(hipmr_kernel* h, int64_t n, void* const* args);
// Whether work put on the stream now may be replayed later.
bool may_be_replayed(void* stream);
int grid_for(long long work_units, int per_block, const LaunchCfg& cfg, int cap);
// geometry stored by the autotuner for (op, combine, neutral, size class of n)
bool tuned_config(hipmr_kernel* h, const char* op, const char* combine, const char* neutral,
                  long long n, hipmr_launch_config* out);
// cfgp with HIPMR_CFG_TUNED: the stored geometry when one exists and resolves,
// else cfgp without the flag (copied into *buf); any other cfgp unchanged
const hipmr_launch_config* apply_tuned(hipmr_kernel* h, const char* op, const char* combine,
                                       const char* neutral, long long n,
                                       const hipmr_launch_config* cfgp, hipmr_launch_config* buf);

// the segmented map-reduce on a given workspace (hipmr_reduce_segmented's
// body; the no-allocation entry point passes its static scratch array)
size_t segmented_workspace(const hipmr_kernel* h, int32_t nseg, int64_t total_n);
hipmr_status reduce_segmented_on(hipmr_kernel* h, const char* combine, const char* neutral,
                                 int32_t nseg, const int64_t* d_offsets, int64_t total_n,
                                 void* const* args, void* d_out, void* workspace,
                                 size_t workspace_bytes, const hipmr_launch_config* cfgp,
                                 void* stream);

// builds the conjugate-gradient kernels (no GPU needed), counting them in *built
hipmr_status cg_selftest(int32_t* built);

// device source of the serving loop's kernels
std::string serve_source(const std::string& prefix);

}  // namespace hipmr
