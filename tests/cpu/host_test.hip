// The library's host side on a stand-in for the HIP runtime: memory is the host's, kernels are written down with their grids and
// arguments and not run (except the copy of logits to the host, which is done here).  usage: host_test SCENARIO
#include "../../include/amusd.h"
#include "../../paper_2410_17375_amd/csrc/amusd_prefill.hip"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

using namespace amusd;

#define CHECK(cond)                                                             \
    do {                                                                        \
        if (!(cond)) {                                                          \
            std::printf("line %d: %s (%s)\n", __LINE__, #cond, amusd_last_error()); \
            std::exit(1);                                                       \
        }                                                                       \
    } while (0)

// ---------------------------------------------------------------- the stand-in
struct Launch {
    std::string name;
    dim3 grid;
    PassArgs pass;
    PrefillArgs prompt;
};
struct Pinned {
    size_t bytes;
    unsigned flags;
};
static std::vector<Launch> launches;
static std::map<void*, Pinned> pinned;
static size_t refuse_pinned = SIZE_MAX;      // blocks of this size and more find no memory
static int copies = 0;                       // hipMemcpy to the host
static int current_device = 0, pinned_device = -1;
static std::map<const void*, std::string>& names() {
    static auto& n = *new std::map<const void*, std::string>();
    return n;
}
static bool has(const std::string& name, const char* kernel) { return name.find(std::to_string(std::strlen(kernel)) + kernel) != std::string::npos; }
static int count(const char* kernel) {
    int n = 0;
    for (const Launch& l : launches) n += has(l.name, kernel);
    return n;
}

extern "C" {
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, uint3*, uint3*, dim3*, dim3*, int*) { names()[host] = name; }
static thread_local struct { dim3 grid, block; size_t lds; hipStream_t stream; } config;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
    config = {grid, block, lds, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
    *grid = config.grid; *block = config.block; *lds = config.lds; *stream = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t) {
    Launch l{names()[f], grid, {}, {}};
    if (has(l.name, "k_accept")) l.pass = *static_cast<PassArgs*>(args[1]);
    if (has(l.name, "k_pf_greedy")) l.prompt = *static_cast<PrefillArgs*>(args[2]);
    if (has(l.name, "k_export")) {
        const size_t bytes = *static_cast<size_t*>(args[4]);
        std::memcpy(*static_cast<char**>(args[0]), *static_cast<const char**>(args[3]), bytes);
        for (size_t c = 0; c * kExportChunk < bytes; ++c) (*static_cast<int**>(args[1]))[c * kExportFlagStep] = *static_cast<int*>(args[2]);
    }
    launches.push_back(l);
    return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t s, hipEvent_t, hipEvent_t, int) {
    return hipLaunchKernel(f, grid, block, args, lds, s);
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t bytes) { return (*p = std::calloc(1, bytes)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned flags) {
    if (bytes >= refuse_pinned) return hipErrorOutOfMemory;
    *p = std::calloc(1, bytes);
    pinned[*p] = Pinned{bytes, flags};
    pinned_device = current_device;
    return hipSuccess;
}
hipError_t hipHostFree(void* p) { pinned.erase(p); std::free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** dev, void* host, unsigned) { *dev = host; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* symbol) { *p = const_cast<void*>(symbol); return hipSuccess; }
hipError_t hipMemcpy(void* dst, const void* src, size_t bytes, hipMemcpyKind kind) {
    copies += kind == hipMemcpyDeviceToHost;
    std::memcpy(dst, src, bytes);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind, hipStream_t) { std::memcpy(dst, src, bytes); return hipSuccess; }
hipError_t hipMemsetAsync(void* dst, int value, size_t bytes, hipStream_t) { std::memset(dst, value, bytes); return hipSuccess; }
hipError_t hipGetDevice(int* device) { *device = current_device; return hipSuccess; }
hipError_t hipSetDevice(int device) { current_device = device; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 2; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) { *p = hipDeviceProp_t{}; p->multiProcessorCount = 256; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
}

static amusd_model* model(amusd_config c) {
    static std::vector<char> zeros(64 << 20);
    amusd_model* m = nullptr;
    CHECK(amusd_model_create(&c, nullptr, &m) == AMUSD_OK);
    for (int id = 0; id < AMUSD_T_COUNT; ++id)
        for (int l = 0; l < (id <= AMUSD_T_FINAL_NORM ? 1 : c.n_layers); ++l) CHECK(amusd_model_set_tensor(m, id, l, zeros.data(), 0) == AMUSD_OK);
    CHECK(amusd_model_finalize(m) == AMUSD_OK);
    return m;
}
static amusd_config tiny(int vocab, int max_ctx) {
    return amusd_config{2, 64, 8, 2, 64, 64, vocab, max_ctx, 16, AMUSD_DTYPE_BF16, 1e4f, 1e-5f, 2};
}
static size_t largest_pinned() {
    size_t n = 0;
    for (const auto& p : pinned) n = std::max(n, p.second.bytes);
    return n;
}

// The pinned block that logits go through is for models that keep logits.
static void logits_block() {
    constexpr int kVocab = 65552;                 // 16 rows are 4 MB and a bit
    amusd_model* m = model(tiny(kVocab, 256));
    std::vector<int32_t> toks(16, 1);
    std::vector<float> out(16 * kVocab, 7.f);
    CHECK(largest_pinned() < 64 << 10);
    CHECK(amusd_prefill(m, toks.data(), 8, nullptr) == AMUSD_OK);
    CHECK(amusd_set_option(m, AMUSD_OPT_KEEP_LOGITS, 0) == AMUSD_OK && largest_pinned() < 64 << 10);
    current_device = 1;                           // the calling thread's; the block is for the model's
    CHECK(amusd_set_option(m, AMUSD_OPT_KEEP_LOGITS, 1) == AMUSD_OK && current_device == 1 && pinned_device == 0);
    CHECK(largest_pinned() >= 4 << 20 && largest_pinned() < (4 << 20) + (64 << 10));
    const size_t blocks = pinned.size();
    for (const auto& p : pinned) CHECK(p.second.bytes < 4 << 20 || p.second.flags == hipHostMallocCoherent);
    CHECK(amusd_set_option(m, AMUSD_OPT_KEEP_LOGITS, 1) == AMUSD_OK && pinned.size() == blocks);
    CHECK(amusd_prefill(m, toks.data(), 16, nullptr) == AMUSD_OK);
    CHECK(amusd_get_logits(m, out.data(), 8) == AMUSD_OK && copies == 1);      // another device's thread: a plain copy
    current_device = 0;
    int32_t n, next;
    CHECK(amusd_verify(m, amusd_kv_len(m), toks.data(), 16, &n, &next) == AMUSD_OK);
    CHECK(amusd_get_logits(m, out.data(), 16) == AMUSD_OK && copies == 1 && count("k_export") == 2);
    for (float x : out) CHECK(x == 0.f);
    CHECK(amusd_model_free(m) == AMUSD_OK);
    refuse_pinned = 1 << 20;                      // no memory for the block: plain copies
    m = model(tiny(kVocab, 256));
    CHECK(amusd_set_option(m, AMUSD_OPT_KEEP_LOGITS, 1) == AMUSD_OK);
    CHECK(amusd_prefill(m, toks.data(), 8, nullptr) == AMUSD_OK);
    CHECK(amusd_get_logits(m, out.data(), 8) == AMUSD_OK && copies == 2 && count("k_export") == 2);
    CHECK(amusd_model_free(m) == AMUSD_OK);
    CHECK(pinned.empty());
}

// Of a prompt's stretches only the last one's logits can be asked for: no other's go to the host.
static void logits_of_stretches() {
    amusd_model* m = model(tiny(512, 6000));
    std::vector<int32_t> toks(5000, 1);
    CHECK(amusd_set_option(m, AMUSD_OPT_KEEP_LOGITS, 1) == AMUSD_OK);
    CHECK(amusd_prefill(m, toks.data(), 5000, nullptr) == AMUSD_OK);
    std::vector<int> sent;
    int last = 0;
    for (const Launch& l : launches)
        if (has(l.name, "k_pf_greedy")) {
            sent.push_back(l.prompt.export_bytes);
            last = l.prompt.n;
            CHECK((int)l.grid.x == (l.prompt.n + 15) / 16 + export_wgs(l.prompt.export_bytes, 512));
        }
    CHECK((sent == std::vector<int>{0, 0, 8 * 512 * 4}) && last < 2048);
    std::vector<float> out(8 * 512);
    CHECK(amusd_get_logits(m, out.data(), 8) == AMUSD_OK && copies == 0 && count("k_export") == 0);
    CHECK(amusd_set_option(m, AMUSD_OPT_PREFILL_WORKSPACE, 0) == AMUSD_OK);      // the same prompt in verify passes
    launches.clear();
    sent.clear();
    CHECK(amusd_kv_rollback(m, 0) == AMUSD_OK && amusd_prefill(m, toks.data(), 19, nullptr) == AMUSD_OK);
    for (const Launch& l : launches)
        if (has(l.name, "k_accept")) sent.push_back(l.pass.export_bytes);
    CHECK((sent == std::vector<int>{0, 0, 3 * 512 * 4}));
    CHECK(amusd_get_logits(m, out.data(), 3) == AMUSD_OK && copies == 0 && count("k_export") == 0);
    CHECK(amusd_model_free(m) == AMUSD_OK);
}

// Workgroups that share tiles write their sums to a buffer: a launch that would go past its end, or past the counters, is refused.
static void shared_sums() {
    DevModel M{};
    M.dtype = AMUSD_DTYPE_BF16;
    M.d = 4096;
    M.F = 14336;
    M.split_down = 2;
    PfTileSet tiles[kPfStages];
    std::vector<int> orders;
    prefill_tile_orders(M, kPfDown, 256, orders, tiles[kPfDown]);
    PrefillBufs T{};
    T.cus = 256;
    const PrefillArgs P{61, 0, 0, 61, 0};
    auto gemm = [&](int shares) { return launch_pf_gemm_v<BF16, kPfDown, PfMid>(M, DevLayer{}, T, tiles, P, nullptr, nullptr, nullptr, shares); };
    T.xch_bytes = (size_t)4096 * 64 * 4 * 16 - 1;          // 64 rows of 4096 columns, 16 slices
    CHECK(gemm(16) == hipErrorInvalidValue && launches.empty());
    CHECK(gemm(2) == hipSuccess && count("k_pf_gemm") == 1 && count("k_pf_add") == 1);
    ++T.xch_bytes;
    CHECK(gemm(16) == hipSuccess && count("k_pf_gemm") == 2 && count("k_pf_add") == 2);
    T.xch_bytes = 0;
    CHECK(gemm(1) == hipSuccess && count("k_pf_gemm") == 3 && count("k_pf_add") == 2);
    auto stream = [&](int shares) { return launch_pf_stream_v<BF16, kPfDown, 4, 2, 4>(M, DevLayer{}, T, tiles, P, nullptr, nullptr, shares); };
    T.xch_bytes = (size_t)4096 * 64 * 4 * 2 - 1;
    CHECK(stream(2) == hipErrorInvalidValue && stream(1) == hipSuccess && count("k_pf_stream") == 1);
    ++T.xch_bytes;
    CHECK(stream(2) == hipSuccess && count("k_pf_stream") == 2);
    PrefillArgs many = P;                                   // more tiles than counters
    many.n = (kPfTickets / 64 + 1) * 32;
    T.xch_bytes = SIZE_MAX;
    CHECK((launch_pf_stream_v<BF16, kPfDown, 4, 2, 4>(M, DevLayer{}, T, tiles, many, nullptr, nullptr, 2) == hipErrorInvalidValue));
}

// Over how many workgroups a prompt's contractions share the K slices of their tiles, against measured times: us a prompt (several layers)
// as it is to be, and with the other number.
static void shares_against_measured_times() {
    struct Point {
        int d, F, q, kv, dtype, split_down, stage, rows, shares, other;
        double us, other_us;
    };
    static const Point points[] = {
        {1024, 4096, 1024, 256, AMUSD_DTYPE_BF16, 1, kPfDown, 600, 2, 1, 910.6, 960.7},     {1024, 4096, 1024, 256, AMUSD_DTYPE_BF16, 1, kPfDown, 1300, 2, 1, 1494.9, 1583.8},
        {2560, 6912, 2048, 512, AMUSD_DTYPE_BF16, 0, kPfDown, 425, 8, 1, 911.5, 963.3},     {3072, 8192, 2048, 512, AMUSD_DTYPE_BF16, 0, kPfDown, 350, 8, 1, 1040.5, 1104.6},
        {5120, 13824, 5120, 1280, AMUSD_DTYPE_BF16, 0, kPfDown, 310, 8, 1, 1634.3, 1711.0}, {4096, 14336, 4096, 1024, AMUSD_DTYPE_BF16, 2, kPfDown, 160, 2, 16, 1119.4, 1127.7},
        {4096, 14336, 4096, 1024, AMUSD_DTYPE_BF16, 2, kPfDown, 1370, 2, 1, 5444.9, 5536.2}, {8192, 8192, 4096, 512, AMUSD_DTYPE_BF16, 0, kPfQKV, 105, 8, 1, 699.3, 707.6},
        {2048, 8192, 2048, 512, AMUSD_DTYPE_FP32, 1, kPfDown, 310, 16, 2, 2160.4, 2337.5},
    };
    for (const Point& p : points) {
        DevModel M{};
        M.dtype = p.dtype;
        M.d = p.d;
        M.F = p.F;
        M.qdim = p.q;
        M.nqkv = p.q + 2 * p.kv;
        M.split_down = p.split_down;
        PfTileSet tiles[kPfStages];
        std::vector<int> orders;
        prefill_tile_orders(M, p.stage, 256, orders, tiles[p.stage]);
        PrefillBufs T{};
        T.cus = 256;
        T.xch_bytes = 2 * kPfShareBytes;
        const int shares = plan_pf_gemm(M, T, tiles, p.rows, p.stage).shares;
        if (shares != p.shares) std::printf("width %d, %d rows: over %d workgroups, not %d (%.0f us), %d: %.0f us\n", p.d, p.rows, shares, p.shares, p.us, p.other, p.other_us);
        CHECK(p.us < p.other_us && shares == p.shares);
    }
}

// A pass launches the same kernels whichever of its stages is timed.
static void timed_stages() {
    for (const int ctx : {40, 700}) {                       // without a merge of chunks, with one
        amusd_model* m = model(tiny(512, 800));
        std::vector<int32_t> toks(ctx, 1);
        std::vector<std::string> plain;
        CHECK(amusd_prefill(m, toks.data(), ctx, nullptr) == AMUSD_OK);
        for (int stage = -1; stage < AMUSD_STAGE_COUNT; ++stage) {
            CHECK(amusd_set_option(m, AMUSD_OPT_TIME_STAGE, stage) == AMUSD_OK);
            launches.clear();
            int32_t n, next;
            CHECK(amusd_verify(m, ctx - 4, toks.data(), 4, &n, &next) == AMUSD_OK);
            std::vector<std::string> now;
            for (const Launch& l : launches) now.push_back(l.name);
            if (stage < 0) plain = now;
            CHECK(now == plain && count("k_attn_merge") == (ctx == 40 ? 0 : 2));
            double ms;
            int64_t timed, bytes;
            if (stage >= 0) CHECK(amusd_stage_time(m, &ms, &timed, &bytes) == AMUSD_OK);
            if (stage == AMUSD_STAGE_ATTENTION) CHECK(timed == 2);
            if (stage == AMUSD_STAGE_ATTN_MERGE) CHECK(timed == count("k_attn_merge") && (timed > 0) == (ms > 0));
        }
        CHECK(amusd_model_free(m) == AMUSD_OK);
    }
}

// Prints the attention kernel that a verify pass takes.  usage: host_test form HEADS KV_HEADS HEAD_DIM CONTEXT ROWS TOKENS [ROWS TOKENS ..],
// a pair for each sequence (16-bit models)
static void form(int argc, char** argv) {
    const int n_seq = (argc - 6) / 2;
    amusd_config c = tiny(512, std::atoi(argv[5]));
    c.n_q_heads = std::atoi(argv[2]);
    c.n_kv_heads = std::atoi(argv[3]);
    c.head_dim = std::atoi(argv[4]);
    c.max_seqs = n_seq;
    amusd_model* m = model(c);
    std::vector<int32_t> toks(c.max_ctx, 1), ids, rows, ctx, accepted(n_seq), next(n_seq);
    for (int i = 0; i < n_seq; ++i) {
        ids.push_back(i);
        rows.push_back(std::atoi(argv[6 + 2 * i]));
        ctx.push_back(std::atoi(argv[7 + 2 * i]));
        CHECK(amusd_seq_prefill(m, i, toks.data(), ctx[i], nullptr) == AMUSD_OK);
    }
    launches.clear();
    CHECK(amusd_verify_batch(m, n_seq, ids.data(), ctx.data(), rows.data(), toks.data(), accepted.data(), next.data()) == AMUSD_OK);
    std::vector<std::string> taken;
    for (const char* k : {"k_attention", "k_attention_g4", "k_attention_g8", "k_attention_packed", "k_attention_whole"})
        if (count(k)) taken.push_back(k);
    CHECK(taken.size() == 1);
    std::printf("%s\n", taken[0].c_str());
}

int main(int argc, char** argv) {
    const std::string scenario = argc > 1 ? argv[1] : "";
    if (scenario == "logits_block") logits_block();
    else if (scenario == "logits_of_stretches") logits_of_stretches();
    else if (scenario == "shared_sums") shared_sums();
    else if (scenario == "shares_against_measured_times") shares_against_measured_times();
    else if (scenario == "timed_stages") timed_stages();
    else if (scenario == "form" && argc >= 8 && argc % 2 == 0) form(argc, argv);
    else return 2;
    std::printf("OK\n");
    return 0;
}
