// Prefix scan of a map (the parallel prefix sums the paper lists among the
// facilities built from the same ingredients as the map-reduce: a map over
// the formal index i, a combine in a and b, its neutral element; section
// "Further Facilities" with section "Map-Reduce").
//
// The array is cut into tiles (see the tile kernel's comment); a tile stays
// in registers from its load to its stores.  Three ways to give a tile the
// fold of everything before it, chosen by size below:
//   one launch        sc1 / sc1s   one tile holds the whole array
//   two launches      scu, scd     tile totals, then every tile folds its
//                                  predecessors' totals itself (input read twice)
//   clear + one pass  scz, scl     tiles publish totals and wait for their
//                                  predecessors' (input read once)
// The order of every combination depends only on n, the alignment head and
// the geometry, so a result is bitwise repeatable.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <atomic>
#include <cctype>
#include <mutex>
#include <new>
#include <set>
#include <string>
#include <vector>

#include "internal.h"

using namespace hipmr;

namespace {

// Tiles and forms by size, from sweeps on MI355X (us per call; float, and
// int32 -> int64 with half the elements per tile):
// - one tile of 1024 threads x 8 sub-tiles where it holds all: one launch
//   instead of two;
// - totals then rescan while a pass over the tiles is short and the second
//   read comes out of the caches: 512 x 8 takes 16.0 / 24.7 at n = 2^23 and
//   34.3 / 49.0 at 2^24, the one-pass form 17.2 / 27.6 and 30.9 / 50.1; every
//   tile folds all earlier totals, so many small tiles cost (256 x 8: 63.7
//   for the 4096 tiles of 2^24 int64), few leave compute units idle (256 x 8:
//   10.8 at 2^22 float);
// - one pass above: large tiles, as each takes a ticket from one counter
//   (about 12 ns per ticket bounds 256 x 4 to 0.80 ms at n = 2^28), and two
//   blocks of 512 threads x 16 sub-tiles (126 registers) fill a compute unit:
//   0.365 ms at n = 2^28 float and 0.302 ms at 2^27 int64, against 0.384 and
//   0.328 for 1024 x 8 and 0.398 / 0.364 for 256 x 16 or 512 x 8.
// A thread holds `per` 32-bit words per sub-tile (its elements of every array
// and of the result); `most` bounds them where spilling costs more than smaller
// tiles do: twelve float arrays of 16384 took 134 us in one tile of 1024 x 8,
// 8.7 in tiles that fit; four arrays 23 and 7.  (Not in the one-pass form,
// where large tiles are the better ones even so: twelve arrays of 2^24 143 us
// against 153 with 8 sub-tiles, 156 with 4.)
struct ScanShape {
    int block, ipt, most;
};
constexpr ScanShape kScanOne = {1024, 8, 80}, kScanSmall = {256, 8, 256}, kScanMid = {512, 8, 128},
                    kScanPass = {512, 16, 0};
// A map or a combine that calls functions is expanded for every element of a
// thread's run: short runs, or the code leaves the instruction cache and the
// functions' temporaries spill.  expf * sinf of 2^26 floats 153 us with these
// against 338; powf of 2^17 9.4 against 24.2; a logarithm of a sum of
// exponentials as the combine, 2^14 floats, 10.5 against 32.5.
constexpr ScanShape kCallsOne = {512, 2, 0}, kCallsSmall = {256, 2, 0}, kCallsMid = {512, 4, 0},
                    kCallsPass = {1024, 4, 0};
constexpr int kScanOwnWords = 128;           // of a geometry the call chose
constexpr long long kScanSmallTiles = 512, kScanFoldTiles = 768;
constexpr long long kScanMinTiles = 64000;   // the workspace holds at least this many totals

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// Bytes per index of the arrays moved in chunks.
int chunk_bytes(const Signature& sig) {
    int b = 0;
    for (auto& a : sig.args)
        if (chunked(a) || a.shifted) b += dtype_size(a.dtype);
    return b;
}

// Whether a combine calls functions that take more than an instruction or two.
bool combine_calls(const char* combine) {
    if (canonical_combine(combine) != Combine::Generic) return false;
    static const std::set<std::string> cheap = {"fabsf", "fabs", "fmaf", "fma", "fmaxf", "fminf", "fmax", "fmin", "max", "min"};
    std::string word;
    for (const char* c = combine; *c; ++c) {
        if (std::isalnum((unsigned char)*c) || *c == '_') {
            word += *c;
        } else if (*c == '(' && !word.empty()) {
            if (!cheap.count(word)) return true;
            word.clear();
        } else if (!std::isspace((unsigned char)*c)) {
            word.clear();
        }
    }
    return false;
}

KernelSpec scan_spec(bool vector, int mode, const LaunchCfg& cfg, bool idx64, const char* combine,
                     const char* neutral) {
    KernelSpec s;
    s.kind = vector ? KernelKind::ScanVector : KernelKind::ScanScalar;
    s.scan_mode = mode;
    s.idx64 = idx64;
    s.block = cfg.block;
    s.ipt = cfg.ipt;
    s.vec = cfg.vec;
    s.nt_loads = cfg.nt_loads;
    s.nt_stores = cfg.nt_stores;
    s.unaligned = cfg.unaligned;
    s.combine = combine;
    s.neutral = neutral;
    return s;
}

// 64-bit words of the one-pass form's ticket counter and published totals:
// tiles, groups of 64, groups of 64 groups.
long long state_words(long long tiles, size_t rs) {
    const long long groups = (tiles + 63) / 64, supers = (groups + 63) / 64;
    return 16 + (tiles + groups + supers) * (long long)(rs / 4);
}

// The current device's word that a scan sets when it gives up a wait: pinned
// host memory, kept for the life of the process.  Null until a scan that may
// wait has allocated it outside a capture (`allocate`).
std::atomic<unsigned>* gave_up_word(bool allocate, void* stream) {
    constexpr int kDevices = 64;
    static std::mutex mu;
    static std::atomic<std::atomic<unsigned>*> words[kDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return nullptr;
    std::atomic<unsigned>* w = words[dev].load(std::memory_order_acquire);
    if (w || !allocate || may_be_replayed(stream)) return w;
    std::lock_guard<std::mutex> lk(mu);
    if ((w = words[dev].load())) return w;
    void* p = nullptr;
    if (hipHostMalloc(&p, sizeof(std::atomic<unsigned>), hipHostMallocDefault) == hipSuccess)
        words[dev].store(w = new (p) std::atomic<unsigned>(0), std::memory_order_release);
    else
        (void)hipGetLastError();
    return w;
}

}  // namespace

extern "C" {

size_t hipmr_scan_workspace_bytes(hipmr_handle h, int64_t n) {
    if (!h || !h->prog.sig.is_reduce || n < 0) return 0;
    const size_t rs = (size_t)dtype_size(h->prog.sig.result);
    return align256((size_t)state_words(kScanMinTiles, rs) * 8);
}

hipmr_status hipmr_scan(hipmr_handle h, const char* combine, const char* neutral, int64_t n,
                        void* const* args, void* out, int32_t exclusive, void* workspace,
                        size_t workspace_bytes, const hipmr_launch_config* cfgp, void* stream) {
    clear_error();
    hipmr_status st = check_args(h, n, args);
    if (st != HIPMR_OK) return st;
    if (!h->prog.sig.is_reduce) return fail(HIPMR_E_MISMATCH, "elementwise handle passed to hipmr_scan");
    if (!combine || !neutral) return fail(HIPMR_E_INVALID, "combine_op and neutral are required");
    if (exclusive != 0 && exclusive != 1) return fail(HIPMR_E_INVALID, "exclusive must be 0 or 1");
    if (n == 0) return HIPMR_OK;
    if (!out) return fail(HIPMR_E_INVALID, "out is NULL");
    if (!workspace || workspace_bytes < hipmr_scan_workspace_bytes(h, n))
        return fail(HIPMR_E_WORKSPACE, "workspace smaller than hipmr_scan_workspace_bytes()");
    workspace_bytes -= align_words(workspace) - (char*)workspace;
    workspace = align_words(workspace);
    // Default chunk: 16 bytes of the narrowest input, but at most 16 bytes of
    // output per lane, so that each store instruction of a wave writes one
    // contiguous run.
    const size_t rs = (size_t)dtype_size(h->prog.sig.result);
    const int dvec = std::min(h->default_vec, std::max(1, 16 / (int)rs));
    LaunchCfg cfg;
    const bool calls = h->map_calls || combine_calls(combine);
    const ScanShape &mid_shape = calls ? kCallsMid : kScanMid, &one_shape = calls ? kCallsOne : kScanOne,
                    &small_shape = calls ? kCallsSmall : kScanSmall, &pass_shape = calls ? kCallsPass : kScanPass;
    st = resolve_cfg(cfgp, mid_shape.block, mid_shape.ipt, dvec, 1, &cfg);
    if (st != HIPMR_OK) return st;

    const long long n64 = n;
    const long long head = vector_head(h, args, &cfg, out, (int)rs);
    const bool vector = head >= 0;
    if (!vector) cfg.vec = 1;
    long long base = head > 0 ? head - cfg.vec : 0;       // tile 0 starts at an aligned element
    auto tiles_of = [&](const LaunchCfg& c) {
        const long long tile = (long long)c.block * c.vec * c.ipt;
        return (n64 - base + tile - 1) / tile;
    };
    const bool own_block = cfgp && cfgp->block, own_ipt = cfgp && cfgp->items_per_thread;
    const int per = std::max(1, cfg.vec * ((int)rs + chunk_bytes(h->prog.sig)) / 4);
    const auto fit = [&](LaunchCfg c, int most) {
        if (own_block || own_ipt) most = kScanOwnWords;
        while (most && c.ipt > 1 && c.ipt * per > most) c.ipt /= 2;
        return c;
    };
    const auto with = [&](const ScanShape& s) {
        LaunchCfg c = cfg;
        if (!own_block) c.block = s.block;
        if (!own_ipt) c.ipt = s.ipt;
        return fit(c, s.most);
    };
    // the one-pass form's tiles are no smaller than its own, whatever the call
    // asked for: every tile costs a ticket (12 ns; 2^26 floats in tiles of
    // 256 x 4 took 219 us, in 64 x 1 772, against 136 in waves of those shapes)
    const auto with_pass = [&] {
        LaunchCfg c = with(pass_shape);
        c.block = std::max(c.block, pass_shape.block);
        c.ipt = std::max(c.ipt, pass_shape.ipt);
        return fit(c, pass_shape.most);
    };
    const bool idx64 = n64 >= (int64_t(1) << 31);
    KernelSpec clear;
    clear.kind = KernelKind::ScanClear;
    const char family = 's' + (own_block ? 1 : 0) + (own_ipt ? 2 : 0);   // the kernels depend on what is the call's own
    st = load_family(h, family, vector, idx64, cfg, combine, neutral, [&] {
        std::vector<KernelSpec> v = {scan_spec(vector, 0, with(one_shape), idx64, combine, neutral),
                                     scan_spec(vector, 3, with_pass(), idx64, combine, neutral), clear};
        for (int mode : {1, 2})
            for (const LaunchCfg& c : {with(small_shape), with(mid_shape)}) v.push_back(scan_spec(vector, mode, c, idx64, combine, neutral));
        return v;
    });
    if (st != HIPMR_OK) return st;
    std::atomic<unsigned>* gave_up = gave_up_word(false, stream);
    if (gave_up && gave_up->load(std::memory_order_relaxed) && gave_up->exchange(0))
        return fail(HIPMR_E_HIP, "an earlier scan on this device gave up waiting for a tile's total: its workspace "
                                 "was written by another call meanwhile, and its outputs are not the scan");
    int mode = 3;
    const LaunchCfg one = with(one_shape), small = with(small_shape), mid = with(mid_shape);
    if (tiles_of(one) == 1) {
        mode = 0;
        cfg = one;
    } else if (tiles_of(small) <= kScanSmallTiles) {
        mode = 2;
        cfg = small;
    } else if (tiles_of(mid) <= kScanFoldTiles) {
        mode = 2;
        cfg = mid;
    } else {
        cfg = with_pass();
    }
    if (mode == 3 && !gave_up) gave_up = gave_up_word(true, stream);
    const long long all = tiles_of(cfg), tile = (long long)cfg.block * cfg.vec * cfg.ipt;
    // tiles whose totals the workspace holds, which one launch takes (below 2^32 threads)
    const long long room = ((long long)(workspace_bytes / 8) - 16) / (long long)(rs / 4);
    const long long at_once = std::min(std::max(room * 4096 / (4096 + 64 + 1) - 2, 1LL), ((1LL << 32) - 1) / cfg.block);
    int tiles = (int)std::min(all, mode == 3 ? at_once : all);
    int flags = exclusive | (cfg.no_wait ? 2 : 0), words = 0;

    CallKernels used;
    void *f_first = nullptr, *f_scan = nullptr;
    st = variant_function(h, scan_spec(vector, mode, cfg, idx64, combine, neutral), &f_scan, &used);
    if (st != HIPMR_OK) return st;
    if (mode == 2) {
        st = variant_function(h, scan_spec(vector, 1, cfg, idx64, combine, neutral), &f_first, &used);
    } else if (mode == 3) {
        st = variant_function(h, clear, &f_first, &used);
    }
    if (st != HIPMR_OK) return st;
    set_last_kernels(h, used);

    std::vector<void*> p;
    if (h->prog.sig.args.empty()) p.push_back(&base);       // hipmr_unused
    for (size_t k = 0; k < h->prog.sig.args.size(); ++k) p.push_back(args[k]);
    long long n_arg = n64;
    p.insert(p.end(), {(void*)&n_arg, (void*)&base, (void*)&tiles, (void*)&workspace, (void*)&out, (void*)&flags, (void*)&gave_up});
    if (mode == 2) st = launch(f_first, (unsigned)tiles, (unsigned)cfg.block, p.data(), stream);
    if (mode != 3) return st != HIPMR_OK ? st : launch(f_scan, (unsigned)tiles, (unsigned)cfg.block, p.data(), stream);
    for (long long done = 0; done < all && st == HIPMR_OK; done += at_once) {
        tiles = (int)std::min(all - done, at_once);
        words = (int)state_words(tiles, rs);
        void* pz[2] = {&workspace, &words};
        st = launch(f_first, (unsigned)((words + 255) / 256), 256, pz, stream);
        if (st != HIPMR_OK) break;
        const int turn = (int)(done / at_once & 1);
        flags = (flags & 3) | (done > 0 ? 4 : 0) | (done + tiles < all ? 8 : 0) | turn << 4;
        st = launch(f_scan, (unsigned)tiles, (unsigned)cfg.block, p.data(), stream);
        base += tiles * tile;
    }
    return st;
}

}  // extern "C"
