// bbe_batch.hip -- batches of uneven Monte-Carlo requests: request
// descriptors and the work list on the device, launch-shape autotuning and
// a captured HIP graph of the whole launch sequence (include/bbe.h).
#include "abi_internal.hpp"

#include <sys/stat.h>
#include <unistd.h>

#include <algorithm>
#include <cstdlib>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

using namespace bbe_abi;

namespace {

// Launch shape.  The tuner chooses among sims_per_item alone; the others are kept
// for shapes that a tuning file holds.
struct Shape {
    int waves_per_block;
    int sims_per_item;  // multiple of 64: one work item = sims_per_item / 64 generations
    int cu_share;       // workgroups per CU: the resident capacity divided by cu_share (1, 2)
};

// Autotune results per (device, size class of the work list), in memory and
// in a JSON file (see tune_cache_path) keyed by the device, the library's
// kernel sources and the size class.
std::mutex g_tune_mu;
std::map<std::pair<int, int>, Shape> g_tuned;
bool g_tune_file_read = false;

struct Group {
    uint32_t first;  // its items: chunks[first .. first + count)
    uint32_t count;
    bool paced;      // the items of races with a time term of R
    // the items of the same requests without shared waves (first and count
    // again where nothing is shared)
    uint32_t alone_first, alone_count;
};

struct Work {
    std::unique_ptr<char[]> bytes;  // the items (of both lists), then the lane table
    size_t size = 0, n_chunks = 0;
    std::vector<Group> groups;
};

// A plan's requests.
struct Requests {
    const bbe::ReqDesc* at;
    size_t n;
    size_t size() const { return n; }
    const bbe::ReqDesc& operator[](size_t i) const { return at[i]; }
    const bbe::ReqDesc* begin() const { return at; }
    const bbe::ReqDesc* end() const { return at + n; }
};

// Hash of a value's bytes: sums of products of neighbouring words, each with a
// constant of its own added (NH of Black, Halevi, Krawczyk, Krovetz and Rogaway's
// UMAC), which the compiler does several at a time.
template <class T>
uint64_t hash_of(const T& v) {
    constexpr size_t words = sizeof(T) / 4;
    static_assert(sizeof(T) % 4 == 0);
    uint32_t w[words + 1];
    std::memcpy(w, &v, sizeof v);
    w[words] = 0;
    uint64_t sum = 0;
    uint32_t k = 0x9E3779B9u;
    for (size_t i = 0; i < words; i += 2, k += 0x9E3779B9u)
        sum += (uint64_t)(w[i] + k) * (w[i + 1] + (k ^ 0x85EBCA6Bu));
    sum *= 0x9E3779B97F4A7C15ull;
    return sum ^ (sum >> 32);
}

// Finds equal ones among numbered values: find(hash, number, equal) gives the
// first number put in for which equal(it) holds, else puts this one in.
class Distinct {
  public:
    explicit Distinct(size_t n) {
        size_t cap = 16;
        while (cap < 2 * n) cap *= 2;
        slots_.assign(cap, UINT32_MAX);
    }
    template <class Equal>
    uint32_t find(uint64_t hash, uint32_t number, const Equal& equal) {
        for (size_t i = hash & (slots_.size() - 1);; i = (i + 1) & (slots_.size() - 1)) {
            if (slots_[i] == UINT32_MAX) return slots_[i] = number;
            if (equal(slots_[i])) return slots_[i];
        }
    }

  private:
    std::vector<uint32_t> slots_;
};

// Expected ticks until the request's simulations end (used only to order
// the work list): remaining distance over a typical free step.
double expected_ticks(const bbe::ReqDesc& r, const bbe::StartState& st) {
    const int n = r.rc.n;
    double lead = 0.0, last = 1e30, fast = 0.0, slow = 1e30;
    for (int k = 0; k < n; ++k) {
        lead = std::max(lead, (double)st.d0[k]);
        last = std::min(last, (double)st.d0[k]);
    }
    for (int c = 0; c < n; ++c) {
        double m = (double)r.rc.elo[c] + 0x1p15 * (double)r.rc.espan16[c];
        fast = std::max(fast, m);
        slow = std::min(slow, m);
    }
    double first = ((double)r.rc.L - lead) / std::max(fast, 1e-30);
    double all = ((double)r.rc.L - last) / std::max(slow, 1e-30);
    double f = n > 1 ? (double)(r.stop_after - 1) / (double)(n - 1) : 0.0;
    return first + f * (all - first);
}

// An item and its place in the order of a launch: plain items first (one
// launch), then paced ones (another), each largest first.
struct Item {
    uint32_t order;
    bbe::Chunk c;
    static uint32_t place(bool paced, double work) {
        const float w = (float)work;  // positive: ordered like its bits
        uint32_t bits;
        std::memcpy(&bits, &w, sizeof bits);
        return (paced ? 0x80000000u : 0u) | (0x7FFFFFFFu - bits);
    }
};

// Puts the items in their order at chunks[at ..]; returns their groups.
std::vector<Group> put_items(std::vector<Item>& items, bbe::Chunk* chunks, size_t at) {
    std::stable_sort(items.begin(), items.end(),
                     [](const Item& a, const Item& b) { return a.order < b.order; });
    std::vector<Group> groups;
    for (const Item& it : items) {
        const bool paced = it.order >> 31;
        if (groups.empty() || groups.back().paced != paced)
            groups.push_back({(uint32_t)at, 0u, paced, 0u, 0u});
        groups.back().count += 1;
        chunks[at++] = it.c;
    }
    return groups;
}

// The work list, and behind it the items of the list without shared waves.
//
// Requests that differ in nothing but their simulations (together[r], the
// first one of r's group, is the same) share waves: what is left of each after
// whole generations of 64 goes to the lane table, request after request.
// That is done where it saves a generation: a shared one takes no longer than
// one of a single request.  10^4 requests of 1 to 200 simulations (37 on
// average) of one race of 20 are 5900 generations instead of 13100; setting
// their states and launching them took 2.54 ms before and 1.20 ms so.
Work build_work(const Requests& reqs, const std::vector<uint32_t>& state_of,
                const std::vector<bbe::StartState>& states,
                const std::vector<uint32_t>& together, int sims_per_item) {
    Work w;
    struct Share {
        uint64_t rests = 0, over = 0;  // requests with a rest, simulations of the rests
        uint64_t at = 0;               // of its next lane in the lane table
        double ticks = -1.0;           // expected
        bool made = false;             // its items of shared waves
        bool shared() const { return (over + 63) / 64 < rests; }
    };
    std::vector<Share> shares(reqs.size());  // at a group's first request
    for (size_t r = 0; r < reqs.size(); ++r) {
        Share& sh = shares[together[r]];
        sh.rests += reqs[r].n_sims % 64 != 0;
        sh.over += reqs[r].n_sims % 64;
        // every request of a group starts from the same state
        if (sh.ticks < 0.0) sh.ticks = expected_ticks(reqs[r], states[state_of[r]]);
    }
    // a group's lanes next to each other
    uint64_t lanes = 0;
    for (Share& sh : shares) {
        sh.at = lanes;
        if (sh.shared()) lanes += sh.over;
    }
    std::vector<Item> items, alone;
    auto add = [&](std::vector<Item>& to, const Share& sh, size_t r, uint64_t first, uint64_t end,
                   uint32_t flags) {
        const bbe::ReqDesc& rq = reqs[r];
        const uint32_t n = (uint32_t)rq.rc.n;
        for (; first < end; first += (uint64_t)sims_per_item) {
            const uint32_t count =
                (uint32_t)std::min<uint64_t>((uint64_t)sims_per_item, end - first);
            // expected competitor-steps: ticks x competitors x simulations
            to.push_back({Item::place(rq.pace.paced != 0, sh.ticks * n * count),
                          {(uint32_t)r, (uint32_t)first, count, n | flags}});
        }
    };
    for (size_t r = 0; r < reqs.size(); ++r) {
        const uint32_t n_sims = reqs[r].n_sims;
        Share& sh = shares[together[r]];
        add(items, sh, r, 0, sh.shared() ? n_sims - n_sims % 64 : n_sims, 0u);
        if (lanes) add(alone, sh, r, 0, n_sims, 0u);
        if (sh.shared() && !sh.made) add(items, sh, r, sh.at, sh.at + sh.over, bbe::kChunkLanes);
        sh.made = true;
    }
    w.n_chunks = items.size() + alone.size();
    w.size = w.n_chunks * sizeof(bbe::Chunk) + lanes * sizeof(bbe::PackLane);
    w.bytes.reset(new char[w.size]);
    bbe::Chunk* chunks = reinterpret_cast<bbe::Chunk*>(w.bytes.get());
    w.groups = put_items(items, chunks, 0);
    // the same launches, one for the plain races and one for the paced
    const std::vector<Group> apart = lanes ? put_items(alone, chunks, items.size()) : w.groups;
    for (size_t g = 0; g < w.groups.size(); ++g) {
        w.groups[g].alone_first = apart[g].first;
        w.groups[g].alone_count = apart[g].count;
    }
    bbe::PackLane* table = reinterpret_cast<bbe::PackLane*>(chunks + w.n_chunks);
    for (size_t r = 0; r < reqs.size(); ++r) {
        const bbe::ReqDesc& rq = reqs[r];
        Share& sh = shares[together[r]];
        if (!sh.shared()) continue;
        for (uint32_t k = rq.n_sims - rq.n_sims % 64; k < rq.n_sims; ++k)
            table[sh.at++] = {(uint32_t)r, rq.sim_begin + k};
    }
    return w;
}

// ---------------------------------------------------------------------------
// Persistent tuning cache.  A JSON file of entries {device, kernels,
// size_class, waves_per_block, sims_per_item, cu_share}, one per line:
// $BBE_TUNE_CACHE if set (empty: no file), else
// $XDG_CACHE_HOME/bbe/tune.json or $HOME/.cache/bbe/tune.json.  An entry
// applies to the device it was tuned on (architecture, name, CU count) and
// to the kernel sources it was tuned with (a hash fixed at build time).
// ---------------------------------------------------------------------------
#ifndef BBE_KERNEL_HASH
#define BBE_KERNEL_HASH "unknown"
#endif

std::string tune_cache_path() {
    if (const char* p = std::getenv("BBE_TUNE_CACHE")) return p;
    if (const char* x = std::getenv("XDG_CACHE_HOME"); x && *x)
        return std::string(x) + "/bbe/tune.json";
    if (const char* h = std::getenv("HOME"); h && *h) return std::string(h) + "/.cache/bbe/tune.json";
    return "";
}

std::string device_key(int dev) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return "unknown";
    char buf[400];
    std::snprintf(buf, sizeof buf, "%s/%s/%d", prop.gcnArchName, prop.name,
                  prop.multiProcessorCount);
    for (char* c = buf; *c; ++c)
        if (*c == '"' || *c == '\\' || (unsigned char)*c < 32) *c = '_';
    return buf;
}

struct TuneEntry {
    std::string device, kernels;
    int size_class;
    Shape shape;
};

std::vector<TuneEntry> read_tune_file(const std::string& path) {
    std::vector<TuneEntry> out;
    FILE* f = path.empty() ? nullptr : std::fopen(path.c_str(), "r");
    if (!f) return out;
    char line[1024];
    while (std::fgets(line, sizeof line, f)) {
        char dev[400], ker[80];
        TuneEntry e;
        if (std::sscanf(line,
                        " {\"device\": \"%399[^\"]\", \"kernels\": \"%79[^\"]\", \"size_class\": %d, "
                        "\"waves_per_block\": %d, \"sims_per_item\": %d, \"cu_share\": %d}",
                        dev, ker, &e.size_class, &e.shape.waves_per_block,
                        &e.shape.sims_per_item, &e.shape.cu_share) == 6) {
            e.device = dev;
            e.kernels = ker;
            out.push_back(e);
        }
    }
    std::fclose(f);
    return out;
}

bool valid_shape(const Shape& s) {
    return (s.waves_per_block == 1 || s.waves_per_block == 2 || s.waves_per_block == 4) &&
           s.sims_per_item >= 64 && s.sims_per_item <= 65536 && s.sims_per_item % 64 == 0 &&
           (s.cu_share == 1 || s.cu_share == 2);
}

// Loads this device's entries for these kernel sources (once per process).
// Call with g_tune_mu held.
void load_tune_cache(int dev) {
    if (g_tune_file_read) return;
    g_tune_file_read = true;
    const std::string me = device_key(dev);
    for (const TuneEntry& e : read_tune_file(tune_cache_path()))
        if (e.device == me && e.kernels == BBE_KERNEL_HASH && valid_shape(e.shape))
            g_tuned[{dev, e.size_class}] = e.shape;
}

// Adds or replaces one entry in the file (best effort: a file that cannot be
// written leaves the in-memory result in place).  Call with g_tune_mu held.
void store_tune_entry(int dev, int size_class, const Shape& sh) {
    const std::string path = tune_cache_path();
    if (path.empty()) return;
    const std::string me = device_key(dev);
    std::vector<TuneEntry> all = read_tune_file(path);
    bool replaced = false;
    for (TuneEntry& e : all)
        if (e.device == me && e.kernels == BBE_KERNEL_HASH && e.size_class == size_class) {
            e.shape = sh;
            replaced = true;
        }
    if (!replaced) all.push_back({me, BBE_KERNEL_HASH, size_class, sh});
    // create the directory one level up (the usual .../bbe/ folder)
    const size_t slash = path.find_last_of('/');
    if (slash != std::string::npos && slash > 0) (void)mkdir(path.substr(0, slash).c_str(), 0755);
    const std::string tmp = path + ".tmp" + std::to_string((long)getpid());
    FILE* f = std::fopen(tmp.c_str(), "w");
    if (!f) return;
    std::fprintf(f, "{\"entries\": [\n");
    for (size_t i = 0; i < all.size(); ++i)
        std::fprintf(f,
                     "  {\"device\": \"%s\", \"kernels\": \"%s\", \"size_class\": %d, "
                     "\"waves_per_block\": %d, \"sims_per_item\": %d, \"cu_share\": %d}%s\n",
                     all[i].device.c_str(), all[i].kernels.c_str(), all[i].size_class,
                     all[i].shape.waves_per_block, all[i].shape.sims_per_item,
                     all[i].shape.cu_share, i + 1 < all.size() ? "," : "");
    std::fprintf(f, "]}\n");
    const bool good = std::fclose(f) == 0;
    if (good) (void)std::rename(tmp.c_str(), path.c_str());
    else (void)std::remove(tmp.c_str());
}

int size_class(size_t n_chunks) {
    int c = 0;
    while (n_chunks > 1) {
        n_chunks >>= 1;
        ++c;
    }
    return c;
}

}  // namespace

struct bbe_batch_plan {
    int device = 0;
    int n_reqs = 0;
    bbe::ReqDesc* d_reqs = nullptr;  // as `table`
    uint32_t* d_queue = nullptr;  // one work-queue head per group
    char* d_work = nullptr;  // the work items (both lists), then the lane table
    size_t work_cap = 0;     // bytes
    size_t n_chunks = 0;     // of both lists
    std::vector<Group> groups;
    std::vector<int> grids;
    uint64_t shared_gens = 0, alone_gens = 0;
    uint64_t slots = 0;  // waves of a launch that are resident at once
    uint32_t k0 = 0, k1 = 0;
    unsigned long long* wins = nullptr;
    double* probs = nullptr;
    unsigned long long* steps = nullptr;
    Shape shape{1, 64, 1};
    int item_sims = 64;  // simulations per work item in use (>= shape.sims_per_item)
    hipStream_t cap_stream = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    std::vector<uint32_t> together;
    // the requests, then (at state_part) whether they run apart (u32, the launch
    // reads it where it runs), each one's state's number from kStateOf on and
    // from states_at on the states; up to `used` bytes
    std::vector<char> table;
    size_t used = 0;
};

namespace {

constexpr size_t kStateOf = 16;
size_t states_at(int n_reqs) {
    return (kStateOf + (size_t)n_reqs * sizeof(uint32_t) + 63) / 64 * 64;
}

size_t state_part(const bbe_batch_plan* p) { return (size_t)p->n_reqs * sizeof(bbe::ReqDesc); }

bbe::ReqDesc* host_reqs(bbe_batch_plan* p) {
    return reinterpret_cast<bbe::ReqDesc*>(p->table.data());
}

Requests requests(bbe_batch_plan* p) { return {host_reqs(p), (size_t)p->n_reqs}; }

const char* d_states(const bbe_batch_plan* p) {
    return reinterpret_cast<const char*>(p->d_reqs + p->n_reqs);
}

bool runs_apart(const bbe_batch_plan* p) {
    uint32_t apart;
    std::memcpy(&apart, p->table.data() + state_part(p), sizeof apart);
    return apart != 0;
}

void keep_states(bbe_batch_plan* p, bool runs_apart, const std::vector<uint32_t>& state_of,
                 const std::vector<bbe::StartState>& states) {
    char* to = p->table.data() + state_part(p);
    const uint32_t apart = runs_apart;
    std::memcpy(to, &apart, sizeof apart);
    std::memcpy(to + kStateOf, state_of.data(), (size_t)p->n_reqs * sizeof(uint32_t));
    const size_t at = states_at(p->n_reqs), bytes = states.size() * sizeof(bbe::StartState);
    std::memcpy(to + at, states.data(), bytes);
    p->used = state_part(p) + at + bytes;
}

hipError_t enqueue(bbe_batch_plan* p, hipStream_t s) {
    hipError_t e;
    if ((e = bbe::launch_zero_u64(p->wins, p->n_reqs * bbe::kMaxN, s)) != hipSuccess) return e;
    if (p->steps && (e = bbe::launch_zero_u64(p->steps, 1, s)) != hipSuccess) return e;
    if ((e = bbe::launch_fill_u32(p->d_queue, 0u, (int)p->groups.size(), s)) != hipSuccess)
        return e;
    const bbe::Chunk* chunks = reinterpret_cast<const bbe::Chunk*>(p->d_work);
    for (size_t g = 0; g < p->groups.size(); ++g) {
        const Group& gr = p->groups[g];
        bbe::BatchArgs a;
        a.reqs = p->d_reqs;
        a.chunks = chunks + gr.first;
        a.n_chunks = gr.count;
        a.alone = chunks + gr.alone_first;
        a.n_alone = gr.alone_count;
        a.apart = reinterpret_cast<const uint32_t*>(d_states(p));
        a.state_of = reinterpret_cast<const uint32_t*>(d_states(p) + kStateOf);
        a.states = reinterpret_cast<const bbe::StartState*>(d_states(p) + states_at(p->n_reqs));
        a.lanes = reinterpret_cast<const bbe::PackLane*>(chunks + p->n_chunks);
        a.queue = p->d_queue + g;
        a.wins = p->wins;
        a.steps = p->steps;
        a.k0 = p->k0;
        a.k1 = p->k1;
        if ((e = bbe::launch_batch_mc(a, p->shape.waves_per_block, p->grids[g], gr.paced, s)) !=
            hipSuccess)
            return e;
    }
    if (p->probs &&
        (e = bbe::launch_batch_probs(p->wins, p->d_reqs, p->n_reqs, p->probs, s)) != hipSuccess)
        return e;
    return hipSuccess;
}

// Generations of a batch: ceil(n_sims / 64) per request.
uint64_t generation_count(const Requests& reqs) {
    uint64_t g = 0;
    for (const bbe::ReqDesc& r : reqs) g += (r.n_sims + 63u) / 64u;
    return g;
}

// The same as build_work makes them, with shared ones counted once.
uint64_t shared_generation_count(const Requests& reqs,
                                 const std::vector<uint32_t>& together) {
    std::vector<uint64_t> over(reqs.size());
    uint64_t g = 0;
    for (size_t r = 0; r < reqs.size(); ++r) {
        g += reqs[r].n_sims / 64u;
        over[together[r]] += reqs[r].n_sims % 64u;
    }
    for (uint64_t o : over) g += (o + 63u) / 64u;
    return g;
}

// Simulations per work item actually used for a shape: the shape's own,
// raised (in whole generations) so that a batch has at most kMaxItems
// items: a batch of very large requests gets fewer, longer items instead of
// a work list of tens of millions.
constexpr uint64_t kMaxItems = 1u << 20;
int item_sims(const Requests& reqs, int sims_per_item) {
    const uint64_t gens = generation_count(reqs);
    const uint64_t min_gens = (gens + kMaxItems - 1) / kMaxItems;
    return (int)std::max<uint64_t>((uint64_t)sims_per_item, 64u * min_gens);
}

// Puts the work lists on the device.
int upload_work(bbe_batch_plan* p, const Shape& sh, const Requests& reqs,
                const std::vector<uint32_t>& state_of,
                const std::vector<bbe::StartState>& states) {
    const int per_item = item_sims(reqs, sh.sims_per_item);
    const Work w = build_work(reqs, state_of, states, p->together, per_item);
    if (w.size > p->work_cap) {
        if (p->d_work) (void)hipFree(p->d_work);
        p->d_work = nullptr;
        p->work_cap = 0;
        if (dev_alloc(&p->d_work, w.size) != hipSuccess)
            return fail(BBE_ENOMEM, "device allocation of the work list failed");
        p->work_cap = w.size;
    }
    hipError_t e = BBE_HIP(hipMemcpy(p->d_work, w.bytes.get(), w.size, hipMemcpyHostToDevice));
    if (e != hipSuccess) return hip_fail(e, "copying the work list");
    p->n_chunks = w.n_chunks;
    p->groups = w.groups;
    p->grids.clear();
    p->shape = sh;
    p->item_sims = per_item;
    const int cus = device_cus();
    for (const Group& g : w.groups) {
        // resident capacity (or a share of it), but no more waves than the
        // launch has items
        long cap = std::max(1L, (long)bbe::batch_blocks_per_cu(sh.waves_per_block, g.paced) /
                                    sh.cu_share) *
                   cus;
        long need = ((long)std::max(g.count, g.alone_count) + sh.waves_per_block - 1) /
                    sh.waves_per_block;
        p->grids.push_back((int)std::max(1L, std::min(cap, need)));
        p->slots = (uint64_t)cap * (uint64_t)sh.waves_per_block;
    }
    return BBE_OK;
}

// Captures clear -> queue reset -> persistent kernel -> probabilities.
int capture(bbe_batch_plan* p) {
    hipError_t e;
    if ((e = BBE_HIP(hipStreamBeginCapture(p->cap_stream, hipStreamCaptureModeThreadLocal))) !=
        hipSuccess)
        return hip_fail(e, "beginning graph capture");
    hipError_t ee = enqueue(p, p->cap_stream);
    e = hipStreamEndCapture(p->cap_stream, &p->graph);
    if (ee != hipSuccess || e != hipSuccess)
        return hip_fail(ee != hipSuccess ? ee : e, "capturing the launch sequence");
    if ((e = BBE_HIP(hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0))) != hipSuccess)
        return hip_fail(e, "instantiating the graph");
    return BBE_OK;
}

// The most runs of equal states that the requests of a group are in.
uint64_t state_runs(const std::vector<uint32_t>& together,
                    const std::vector<uint32_t>& state_of) {
    std::vector<uint32_t> last(together.size(), UINT32_MAX), runs(together.size());
    uint32_t most = 1;
    for (size_t r = 0; r < together.size(); ++r) {
        const uint32_t g = together[r];
        if (last[g] == state_of[r]) continue;
        last[g] = state_of[r];
        most = std::max(most, ++runs[g]);
    }
    return most;
}

// Whether the plan's requests should run apart, their states given.  A shared
// wave goes through its lanes' states one after the other, so with `runs` of
// them a launch may take as long as `runs` launches of one state: of one
// generation for as many waves as are resident, and in proportion from there
// on.  Requests of one race of 20 a third of the way on, us (shared / apart): 64
// of one simulation in 2 states 900 / 351, in 64 states 16800 / 336; 300 of 7 in
// 2 states 891 / 417.
bool better_apart(const bbe_batch_plan* p, const std::vector<uint32_t>& state_of) {
    if (p->shared_gens == p->alone_gens) return false;
    return state_runs(p->together, state_of) * std::max(p->shared_gens, p->slots) >
           std::max(p->alone_gens, p->slots);
}

void destroy(bbe_batch_plan* p) {
    if (!p) return;
    if (p->d_reqs || p->d_queue) (void)hipDeviceSynchronize();
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    if (p->cap_stream) (void)hipStreamDestroy(p->cap_stream);
    if (p->d_reqs) (void)hipFree(p->d_reqs);
    if (p->d_queue) (void)hipFree(p->d_queue);
    if (p->d_work) (void)hipFree(p->d_work);
    delete p;
}

// A request's descriptor (its bytes are set throughout, so that equal ones
// compare equal).
void fill_desc(const bbe_request& q, bbe::ReqDesc& d) {
    std::memset(&d, 0, sizeof d);
    d.rc = q.race->rc;
    d.pace = q.race->pace;
    d.request = q.request;
    d.sim_begin = q.sim_begin;
    d.n_sims = q.n_sims;
    d.stop_after = q.stop_after == 0 ? q.race->n : q.stop_after;
}

// Whether state b of n competitors equals state a, which has been validated.
bool same_state(const bbe_state* a, const bbe_state* b, int n) {
    if (!a || !b) return a == b;
    if (a->tick != b->tick || !b->pos || !b->prev_step) return false;
    const size_t bytes = n * sizeof(float);
    return (a->pos == b->pos || std::memcmp(a->pos, b->pos, bytes) == 0) &&
           (a->prev_step == b->prev_step ||
            std::memcmp(a->prev_step, b->prev_step, bytes) == 0);
}

}  // namespace

namespace {

// Makes plan p for the requests; the caller destroys it where this fails.
int make_plan(bbe_batch_plan* p, const bbe_request* reqs, int n_reqs, uint64_t seed,
              uint64_t* win_counts, double* probs, uint64_t* step_count, unsigned flags,
              void* stream) {
    p->n_reqs = n_reqs;
    p->table.resize((size_t)n_reqs * (sizeof(bbe::ReqDesc) + sizeof(bbe::StartState)) +
                    states_at(n_reqs));
    bbe::ReqDesc* descs = host_reqs(p);
    p->together.resize(n_reqs);
    std::vector<uint32_t> state_of(n_reqs);
    std::vector<bbe::StartState> states;
    Distinct same_states((size_t)n_reqs), groups((size_t)n_reqs);
    for (int i = 0; i < n_reqs; ++i) {
        const bbe_request& q = reqs[i];
        // a row of requests of one race from one state is looked at once
        const bool again = i > 0 && q.race == reqs[i - 1].race;
        int rc = BBE_OK;
        if (again && same_state(reqs[i - 1].state, q.state, q.race->n)) {
            state_of[i] = state_of[i - 1];
        } else {
            bbe::StartState st;
            std::memset(&st, 0, sizeof st);
            rc = q.race ? check_state(q.race, q.state, st.d0, st.s0, st.id0, &st.t0)
                        : fail(BBE_EINVAL, "request %d: race is NULL", i);
            if (rc == BBE_OK) {
                const uint32_t at = (uint32_t)states.size();
                state_of[i] = same_states.find(hash_of(st), at, [&](uint32_t k) {
                    return std::memcmp(&states[k], &st, sizeof st) == 0;
                });
                if (state_of[i] == at) states.push_back(st);
            } else if (q.race) rc = fail(rc, "request %d: %s", i, g_err.c_str());
        }
        if (rc != BBE_OK) {
                return rc;
        }
        if (q.n_sims == 0) {
                return fail(BBE_EINVAL, "request %d: n_sims must be >= 1", i);
        }
        if ((uint64_t)q.sim_begin + q.n_sims > 0x100000000ull) {
                return fail(BBE_EINVAL, "request %d: sim_begin + n_sims exceeds 2^32", i);
        }
        if (q.stop_after < 0 || q.stop_after > q.race->n) {
                return fail(BBE_EINVAL, "request %d: stop_after = %d outside 0..%d", i,
                        q.stop_after, q.race->n);
        }
        bbe::ReqDesc& d = descs[i];
        fill_desc(q, d);
        if (again && state_of[i] == state_of[i - 1] &&
            d.stop_after == descs[i - 1].stop_after) {
            p->together[i] = p->together[i - 1];
            continue;
        }
        const uint64_t hash = hash_of(d.rc) + 31u * hash_of(d.pace) +
                              ((uint64_t)state_of[i] << 5) + (uint64_t)d.stop_after;
        p->together[i] = groups.find(hash, (uint32_t)i, [&](uint32_t k) {
            return state_of[k] == state_of[i] && descs[k].stop_after == d.stop_after &&
                   std::memcmp(&descs[k].rc, &d.rc, sizeof d.rc) == 0 &&
                   std::memcmp(&descs[k].pace, &d.pace, sizeof d.pace) == 0;
        });
    }
    keep_states(p, false, state_of, states);
    p->k0 = (uint32_t)seed;
    p->k1 = (uint32_t)(seed >> 32);
    p->wins = reinterpret_cast<unsigned long long*>(win_counts);
    p->probs = probs;
    p->steps = reinterpret_cast<unsigned long long*>(step_count);
    (void)hipGetDevice(&p->device);

    hipError_t e;
    if (dev_alloc(&p->d_reqs, p->table.size()) != hipSuccess ||
        dev_alloc(&p->d_queue, sizeof(uint32_t) * bbe::kMaxN) != hipSuccess) {
        return fail(BBE_ENOMEM, "device allocation of the request table failed");
    }
    if ((e = BBE_HIP(hipMemcpy(p->d_reqs, p->table.data(), p->used, hipMemcpyHostToDevice))) !=
        hipSuccess) {
        return hip_fail(e, "copying the request table");
    }
    if ((e = BBE_HIP(hipStreamCreateWithFlags(&p->cap_stream, hipStreamNonBlocking))) !=
        hipSuccess) {
        return hip_fail(e, "creating the capture stream");
    }
    hipStream_t s = static_cast<hipStream_t>(stream);

    // Launch shape: tuned on this batch, or from the cache, or the default.
    Shape best{1, 64, 1};
    p->alone_gens = generation_count(requests(p));
    p->shared_gens = shared_generation_count(requests(p), p->together);
    const uint64_t work = p->shared_gens;
    std::pair<int, int> key{p->device, size_class(work)};
    bool have = false;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        load_tune_cache(p->device);
        auto it = g_tuned.find(key);
        if (it != g_tuned.end()) {
            best = it->second;
            have = true;
        }
    }
    if ((flags & BBE_PLAN_AUTOTUNE) && !have) {
        // One wave per workgroup and one generation per item are at least as
        // good as anything else (4096 waves are resident; us, items of 64 and
        // of 128 simulations, then half the workgroups: 5806 items 1280, 1710,
        // 1750; 8192 items 8110, 10820, 9480; 140000 items 16300, 16380, 25100;
        // 4 waves per workgroup within 2%), except that with several items
        // for each resident wave longer ones can end more evenly (22400 items
        // 15.5, 14.5 ms): only there is there something to try.
        std::vector<Shape> cands = {{1, 64, 1}};
        if (work >= 4096u * 4u) cands.push_back({1, 128, 1});
        // Candidates are timed on the batch itself, or -- for a batch of
        // more than kTuneGens generations -- on the same requests with their
        // simulation counts scaled down to about that much work.
        constexpr uint64_t kTuneGens = 1u << 16;
        std::vector<bbe::ReqDesc> tune(descs, descs + n_reqs);
        const uint64_t gens = p->alone_gens;
        if (gens > kTuneGens)
            for (bbe::ReqDesc& r : tune)
                r.n_sims = (uint32_t)std::max<uint64_t>(1u, (uint64_t)r.n_sims * kTuneGens / gens);
        float best_ms = 1e30f;
        hipEvent_t ev0, ev1;
        (void)hipEventCreate(&ev0);
        (void)hipEventCreate(&ev1);
        if (cands.size() < 2) cands.clear();  // nothing to compare
        for (const Shape& c : cands) {
            int rc = upload_work(p, c, {tune.data(), tune.size()}, state_of, states);
            if (rc != BBE_OK) {
                (void)hipEventDestroy(ev0);
                (void)hipEventDestroy(ev1);
                        return rc;
            }
            float ms_min = 1e30f;
            bool okc = true;
            for (int rep = 0; rep < 4 && okc; ++rep) {
                (void)hipEventRecord(ev0, s);
                okc = enqueue(p, s) == hipSuccess;
                (void)hipEventRecord(ev1, s);
                (void)hipEventSynchronize(ev1);
                float ms = 0.0f;
                (void)hipEventElapsedTime(&ms, ev0, ev1);
                if (rep > 0) ms_min = std::min(ms_min, ms);  // first run warms up
            }
            if (okc && ms_min < best_ms) {
                best_ms = ms_min;
                best = c;
            }
        }
        (void)hipEventDestroy(ev0);
        (void)hipEventDestroy(ev1);
        std::lock_guard<std::mutex> lk(g_tune_mu);
        g_tuned[key] = best;
        store_tune_entry(p->device, key.second, best);
    }
    int rc = upload_work(p, best, requests(p), state_of, states);
    if (rc == BBE_OK) rc = capture(p);
    if (rc != BBE_OK) {
        return rc;
    }

    if ((e = hipStreamSynchronize(s)) != hipSuccess) {
        return hip_fail(e, "synchronizing after plan set-up");
    }
    return BBE_OK;
}

// Gives the plan's requests new states.
int point_plan(bbe_batch_plan* plan, const bbe_state* states, void* stream) {
    const int n_reqs = plan->n_reqs;
    // validate every state before touching the plan; a request in the state of
    // the one before it in its group shares that one's entry
    std::vector<uint32_t> state_of(n_reqs), before(n_reqs, UINT32_MAX);
    std::vector<bbe::StartState> distinct;
    distinct.reserve(n_reqs);
    for (int r = 0; r < n_reqs; ++r) {
        const bbe::ReqDesc& q = requests(plan)[r];
        uint32_t& b = before[plan->together[r]];
        if (b != UINT32_MAX && same_state(&states[b], &states[r], q.rc.n)) {
            state_of[r] = state_of[b];
        } else {
            state_of[r] = (uint32_t)distinct.size();
            distinct.emplace_back();
            bbe::StartState& st = distinct.back();
            int rc = check_state(q.rc.n, q.rc.L, &states[r], st.d0, st.s0, st.id0, &st.t0);
            if (rc != BBE_OK) return fail(rc, "request %d: %s", r, g_err.c_str());
        }
        b = (uint32_t)r;
    }
    keep_states(plan, better_apart(plan, state_of), state_of, distinct);
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    (void)hipStreamIsCapturing(s, &cap);
    // ordered after earlier launches on `stream`; the pageable source is
    // consumed before the call returns.  A copy that a graph records takes the
    // whole table, which may hold more states when the graph runs.
    const size_t from = state_part(plan);
    const size_t to = cap == hipStreamCaptureStatusNone ? plan->used : plan->table.size();
    hipError_t e = BBE_HIP(hipMemcpyAsync(plan->d_reqs + n_reqs, plan->table.data() + from,
                                          to - from, hipMemcpyHostToDevice, s));
    if (e != hipSuccess) return hip_fail(e, "copying the request table");
    return ok();
}

}  // namespace

BBE_API int bbe_batch_plan_create(const bbe_request* reqs, int n_reqs, uint64_t seed,
                                  uint64_t* win_counts, double* probs, uint64_t* step_count,
                                  unsigned flags, void* stream, bbe_batch_plan** out) {
    if (!out) return fail(BBE_EINVAL, "out is NULL");
    *out = nullptr;
    if (!reqs || n_reqs < 1) return fail(BBE_EINVAL, "need n_reqs >= 1 requests");
    if (!win_counts) return fail(BBE_EINVAL, "win_counts is NULL");
    bbe_batch_plan* p = new (std::nothrow) bbe_batch_plan();
    if (!p) return fail(BBE_ENOMEM, "out of host memory");
    const int rc = guarded([&] {
        return make_plan(p, reqs, n_reqs, seed, win_counts, probs, step_count, flags, stream);
    });
    if (rc != BBE_OK) {
        destroy(p);
        return rc;
    }
    *out = p;
    return ok();
}

BBE_API int bbe_batch_plan_launch(bbe_batch_plan* plan, void* stream) {
    if (!plan || !plan->exec) return fail(BBE_EINVAL, "plan is NULL");
    hipError_t e = BBE_HIP(hipGraphLaunch(plan->exec, static_cast<hipStream_t>(stream)));
    if (e != hipSuccess) return hip_fail(e, "launching the plan graph");
    return ok();
}

BBE_API int bbe_batch_plan_set_states(bbe_batch_plan* plan, const bbe_state* states,
                                      void* stream) {
    if (!plan || !plan->exec) return fail(BBE_EINVAL, "plan is NULL");
    if (!states) return fail(BBE_EINVAL, "states is NULL");
    return guarded([&] { return point_plan(plan, states, stream); });
}

BBE_API int bbe_batch_plan_info(const bbe_batch_plan* plan, int* waves_per_block, int* grid,
                                int* sims_per_item, int* n_items) {
    if (!plan) return fail(BBE_EINVAL, "plan is NULL");
    if (waves_per_block) *waves_per_block = plan->shape.waves_per_block;
    if (grid) {
        int g = 0;
        for (int x : plan->grids) g = std::max(g, x);
        *grid = g;
    }
    if (sims_per_item) *sims_per_item = plan->item_sims;
    if (n_items) {
        *n_items = 0;
        for (const Group& g : plan->groups)
            *n_items += (int)(runs_apart(plan) ? g.alone_count : g.count);
    }
    return ok();
}

BBE_API void bbe_batch_plan_free(bbe_batch_plan* plan) { destroy(plan); }

namespace {

// The record of one request of an in-play state batch for the kernel, at most
// kPrefixWords words; *words of them.
int put_prefix(const bbe_request& q, uint32_t sim, float target, int idx, uint32_t* w,
               uint32_t* words) {
    if (!q.race) return fail(BBE_EINVAL, "request %d: race is NULL", idx);
    const int n = q.race->n;
    float d[BBE_MAX_COMPETITORS], s[BBE_MAX_COMPETITORS];
    bbe::PrefixHead h;
    int rc = check_values(n, q.race->L, q.state, d, s, &h.t0);
    if (rc != BBE_OK) return fail(rc, "request %d: %s", idx, g_err.c_str());
    if (!std::isfinite(target) || !(target < q.race->L))
        return fail(BBE_EINVAL, "request %d: target must be finite and < track length", idx);
    h.n = (uint32_t)n | (q.race->pace.paced ? bbe::kPrefixPaced : 0u) |
          (q.state ? bbe::kPrefixState : 0u);
    h.request = q.request;
    h.sim = sim;
    h.target = target;
    h.L = q.race->L;
    uint32_t* to = w;
    std::memcpy(to, &h, sizeof h);
    to += sizeof h / 4;
    auto put = [&](const float* v) {
        std::memcpy(to, v, n * sizeof(float));
        to += n;
    };
    const bbe::RaceConst& r = q.race->rc;
    for (const float* v : {r.elo, r.espan16, r.alpha, r.beta, r.theta}) put(v);
    if (q.race->pace.paced)
        for (const float* v : {q.race->pace.gamma, q.race->pace.tau}) put(v);
    if (q.state)
        for (const float* v : {d, s}) put(v);
    *words = (uint32_t)(to - w);
    return BBE_OK;
}

}  // namespace

// The host's part counts most (16384 requests with 5 to 20 competitors:
// 1.95 ms, 0.40 of them GPU time, with whole 850-byte descriptors; 0.93 ms with
// records of what the kernel reads, 260 bytes on average, and the races, which
// lie apart from each other in memory, fetched ahead).
BBE_API int bbe_prefix_batch(const bbe_request* reqs, const uint32_t* sims, const float* targets,
                             int n, uint64_t seed, uint32_t* tick_out, float* pos_out,
                             float* prev_out, void* stream) {
    if (!reqs || !sims || !targets || n < 1) return fail(BBE_EINVAL, "bad batch arguments");
    if (!tick_out || !pos_out || !prev_out) return fail(BBE_EINVAL, "NULL output");
    // where each record begins (u64[n]), then the records
    const size_t head = (size_t)n * sizeof(uint64_t);
    std::unique_ptr<char[]> h(new (std::nothrow)
                                  char[head + (size_t)n * bbe::kPrefixWords * sizeof(uint32_t)]);
    if (!h) return fail(BBE_ENOMEM, "out of host memory");
    uint64_t* at = reinterpret_cast<uint64_t*>(h.get());
    uint32_t* records = reinterpret_cast<uint32_t*>(h.get() + head);
    uint64_t used = 0;
    constexpr int kAhead = 6;
    for (int i = 0; i < n; ++i) {
        if (i + kAhead < n && reqs[i + kAhead].race) {
            const bbe_race* r = reqs[i + kAhead].race;
            __builtin_prefetch(r);
            for (size_t b = 0; b < sizeof r->rc; b += 64)
                __builtin_prefetch(reinterpret_cast<const char*>(&r->rc) + b);
            __builtin_prefetch(&r->pace.paced);
        }
        uint32_t words;
        int rc = put_prefix(reqs[i], sims[i], targets[i], i, records + used, &words);
        if (rc != BBE_OK) return rc;
        at[i] = used;
        used += words;
    }
    const size_t bytes = head + used * sizeof(uint32_t);
    char* d = nullptr;
    if (dev_alloc(&d, bytes) != hipSuccess) return fail(BBE_ENOMEM, "device allocation failed");
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e = BBE_HIP(hipMemcpyAsync(d, h.get(), bytes, hipMemcpyHostToDevice, s));
    if (e == hipSuccess)
        e = BBE_HIP(bbe::launch_prefix_batch(reinterpret_cast<const uint32_t*>(d + head),
                                             reinterpret_cast<const uint64_t*>(d), n,
                                             (uint32_t)seed, (uint32_t)(seed >> 32), tick_out,
                                             pos_out, prev_out, s));
    hipError_t e2 = hipStreamSynchronize(s);
    (void)hipFree(d);
    if (e != hipSuccess) return hip_fail(e, "in-play state batch");
    if (e2 != hipSuccess) return hip_fail(e2, "in-play state batch");
    return ok();
}

// ---------------------------------------------------------------------------
// bbe_prefix_batch without allocations: the requests' records go to a
// fixed device array instead of a per-call hipMalloc.  The array exists once
// per GPU for the life of the process; host code reaches it only through
// the address hipGetSymbolAddress returns on that GPU (the array's own name
// is a host-side stand-in there).
// ---------------------------------------------------------------------------
static __device__ __align__(256) uint32_t scratch[BBE_PREFIX_NOALLOC_MAX * bbe::kPrefixWords];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint32_t* g_scratch_ptr[kMaxDevices] = {};

// Address of the current GPU's copy of `scratch`, looked up once per GPU
// with that GPU current.
int scratch_on_current_device(uint32_t** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(BBE_EDEVICE, "device %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "looking up the static workspace");
        g_scratch_ptr[dev] = static_cast<uint32_t*>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return BBE_OK;
}

}  // namespace

BBE_API int bbe_prefix_batch_noalloc(const bbe_request* reqs, const uint32_t* sims,
                                     const float* targets, int n, uint64_t seed,
                                     uint32_t* tick_out, float* pos_out, float* prev_out,
                                     void* stream) {
    if (!reqs || !sims || !targets || n < 1) return fail(BBE_EINVAL, "bad batch arguments");
    if (n > BBE_PREFIX_NOALLOC_MAX)
        return fail(BBE_EINVAL, "n = %d exceeds the static workspace of %d requests", n,
                    BBE_PREFIX_NOALLOC_MAX);
    if (!tick_out || !pos_out || !prev_out) return fail(BBE_EINVAL, "NULL output");
    uint32_t* d = nullptr;
    int rc = scratch_on_current_device(&d);
    if (rc != BBE_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // records staged through a fixed host block, one piece at a time
    constexpr int kPiece = 32;
    uint32_t h[kPiece * bbe::kPrefixWords] = {};
    for (int i0 = 0; i0 < n; i0 += kPiece) {
        const int m = std::min(kPiece, n - i0);
        for (int j = 0; j < m; ++j) {
            uint32_t words;
            rc = put_prefix(reqs[i0 + j], sims[i0 + j], targets[i0 + j], i0 + j,
                            h + j * bbe::kPrefixWords, &words);
            if (rc != BBE_OK) return rc;  // nothing launched yet; earlier pieces are unused
        }
        hipError_t e = BBE_HIP(hipMemcpyAsync(d + i0 * bbe::kPrefixWords, h,
                                              m * bbe::kPrefixWords * sizeof(uint32_t),
                                              hipMemcpyHostToDevice, s));
        if (e == hipSuccess) e = hipStreamSynchronize(s);  // h is reused by the next piece
        if (e != hipSuccess) return hip_fail(e, "staging the request descriptors");
    }
    hipError_t e =
        BBE_HIP(bbe::launch_prefix_batch(d, nullptr, n, (uint32_t)seed, (uint32_t)(seed >> 32),
                                         tick_out, pos_out, prev_out, s));
    hipError_t e2 = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "in-play state batch");
    if (e2 != hipSuccess) return hip_fail(e2, "in-play state batch");
    return ok();
}
