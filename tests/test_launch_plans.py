"""Which kernels a batch call launches, checked on the host: the built library with HIP's launch entry points replaced by a log.  Nothing runs on
a device and no operand's memory is read, so operands of any size can be planned."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <dlfcn.h>
#include <map>
#include <string>
#include <vector>
#include "mor.h"

// ---- what the library calls of HIP
struct Dim3 { uint32_t x, y, z; };
struct Launch { std::string name; int second; };      // `second`: the first word of the second argument, where that is a table that begins with its length
static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static std::vector<Launch> log_;
static Dim3 call_grid, call_block;
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) { names()[host] = device; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t, void*) { call_grid = grid; call_block = block; return 0; }
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) { *grid = call_grid; *block = call_block; *lds = 0; *stream = nullptr; return 0; }
int hipLaunchKernel(const void* f, Dim3, Dim3, void** args, size_t, void*) {
    const std::string& n = names()[f];
    const bool table = n.find("15k_tensor_streamI") != std::string::npos || n.find("k_tensor_finish_") != std::string::npos;
    log_.push_back({n, table ? *static_cast<const int*>(args[1]) : 0});
    return 0;
}
int hipGetLastError() { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = nullptr; return 1; }
int hipEventRecord(void*, void*) { return 0; }
}

struct Op { int gran; int64_t rows, cols, pad; bool stats; int scaling = MOR_SCALE_FP32_AMAX, scope = MOR_SCOPE_PARTITION; bool fake = false; };
static size_t (*ws_bytes)(const mor_batch_item*, int32_t);
static mor_status (*batch)(const mor_batch_item*, int32_t, float, void*, size_t, void*, mor_profile*);

static mor_status run(const std::vector<Op>& ops) {
    uintptr_t next = uintptr_t(1) << 40;                   // addresses of operands: aligned, apart, never read
    auto at = [&] { next += uintptr_t(1) << 38; return reinterpret_cast<void*>(next); };
    std::vector<mor_batch_item> items(ops.size());
    for (size_t i = 0; i < ops.size(); ++i) {
        const Op& o = ops[i];
        mor_batch_item& it = items[i];
        memset(&it, 0, sizeof it);
        it.params.rows = o.rows; it.params.cols = o.cols; it.params.ld = o.cols + o.pad;
        it.params.granularity = o.gran; it.params.scope = o.scope; it.params.criterion = MOR_CRIT_MEAN_REL_ERR;
        it.params.formats = MOR_FMT_E4M3 | MOR_FMT_BF16; it.params.scaling = o.scaling; it.params.threshold = 0.045f;
        it.x = static_cast<const uint16_t*>(at());
        mor_outputs& u = it.out;
        if (!o.fake) {
            u.fp8 = static_cast<uint8_t*>(at()); u.ld_fp8 = o.cols; u.bf16 = static_cast<uint16_t*>(at()); u.ld_bf16 = o.cols;
        } else { it.fake_y = static_cast<uint16_t*>(at()); it.ld_fake_y = o.cols; }
        u.scale = static_cast<float*>(at()); u.amax = static_cast<float*>(at()); u.err_sum = static_cast<float*>(at());
        u.nnz = static_cast<uint32_t*>(at()); u.mask = static_cast<uint8_t*>(at());
        if (o.scaling != MOR_SCALE_FP32_AMAX) { u.scale_e8m0 = static_cast<uint8_t*>(at()); u.group_mantissa = static_cast<uint32_t*>(at()); }
        if (o.stats) it.stats = static_cast<mor_stats*>(at());
    }
    log_.clear();
    const size_t bytes = ws_bytes(items.data(), (int32_t)items.size());
    return batch(items.data(), (int32_t)items.size(), 1e-5f, at(), bytes, nullptr, nullptr);
}
static bool is(const Launch& l, const char* part) { return l.name.find(part) != std::string::npos; }
static int count(const char* part) { int n = 0; for (const Launch& l : log_) n += is(l, part); return n; }
// A launch that clears the words of streamed operands is followed by the passes that use them, those of per-tensor operands by the finish pass.
static bool passes_follow() {
    for (size_t i = 0; i < log_.size(); ++i) {
        auto then = [&](size_t k, const char* part) { return i + k < log_.size() && is(log_[i + k], part); };
        if (is(log_[i], "k_tensor_stream_clear") && !(then(1, "15k_tensor_streamI") && then(2, "k_tensor_finish_"))) return false;
        if (is(log_[i], "14k_stream_clear") && !then(1, "k_team_streamI")) return false;
        if (is(log_[i], "k_pair_clear") && !then(1, "k_pair_firstI")) return false;
        if (is(log_[i], "k_pair_firstI") && !then(1, "k_pair_secondI")) return false;
        // (columns that share a launch with rows form their scales in it)
        if (is(log_[i], "k_pair_secondI") && !(i && (is(log_[i - 1], "k_pair_firstI") || is(log_[i - 1], "k_col_groupI")))) return false;
    }
    return true;
}
static const int T = MOR_GRAN_TENSOR, B128 = MOR_GRAN_BLOCK_128x128, S = MOR_GRAN_SUB_1x128, B64 = MOR_GRAN_BLOCK_64x64;

// Per-tensor operands with padded rows take 128 x 128 blocks along, also without a 1 x 128 operand in a form that could share their launch.
static bool padded_with_blocks() {
    for (int stats = 0; stats < 2; ++stats)
        for (int subs = 0; subs < 3; ++subs) {
            std::vector<Op> ops{{T, 4200, 2048, 2048, stats != 0}, {B128, 1024, 1024, 0, stats != 0}};
            for (int k = 0; k < subs; ++k) ops.push_back({S, 1024, 1024, 0, stats != 0});
            if (run(ops) != MOR_OK || !passes_follow()) return false;
            if (count("15k_tensor_streamI") != 1 || count("k_tensor_finish_fillI") != 1 || count("k_tensor_finish_groupI") != 0) return false;
        }
    return true;
}
// The finish pass of operands that nothing goes along with is the one without the others' statistics.
static bool nothing_along() {
    for (int64_t rows = 256; rows <= 8192; rows *= 2)
        for (int64_t pad = 0; pad <= 8; pad += 8) {
            if (run({{T, rows, 4096, pad, true}, {T, rows, 2048, pad, true}, {B64, 256, 256, 0, true}}) != MOR_OK || !passes_follow()) return false;
            if (count("k_tensor_finish_fillI") != 0 || count("k_tensor_finish_groupI") != 1) return false;
        }
    return true;
}
// A small per-tensor operand alone keeps its own two launches beside others, unless there are statistics of those to take along.
static bool small_alone() {
    for (int64_t pad = 0; pad <= 8; pad += 8)
        for (int counted = 0; counted < 4; ++counted)
            for (int gran : {S, B128})
                for (int64_t rows : {64, 465, 2048, 2560}) {
                    if (run({{T, rows, 4096, pad, (counted & 1) != 0}, {gran, 128, 1024, pad, (counted & 2) != 0}}) != MOR_OK || !passes_follow()) return false;
                    const int want = counted / 2 || rows > 2048 ? 1 : 0;
                    if (count("15k_tensor_streamI") != want || count("k_tensor_quant_oneI") != 1 - want) return false;
                }
    return true;
}
// Blocks go along with passes of some hundred tiles where that saves their launch, not where it stays for blocks that have a pre-pass.
static bool blocks_that_stay() {
    for (int scaling : {MOR_SCALE_FP32_AMAX, MOR_SCALE_GAM}) {
        const int want = scaling == MOR_SCALE_GAM ? 0 : 1;
        if (run({{T, 3681, 1336, 0, true}, {T, 2059, 1760, 0, true}, {B128, 1408, 1280, 0, false}, {B128, 2304, 384, 0, false, scaling}}) != MOR_OK || !passes_follow()) return false;
        if (count("15k_tensor_streamI") != want || count("k_team_groupI") != 1 - want) return false;
    }
    return true;
}
// Statistics that the finish pass takes: at most twelve operands' in its table, also where a dense 1 x 128 operand cannot share the launch.
static bool statistics_fit() {
    for (int64_t pad = 0; pad <= 2048; pad += 2048)
        for (int subs = 0; subs < 3; ++subs)
            for (int others = 8; others < 14; ++others) {
                std::vector<Op> ops{{T, 1024, 2048, pad, true}, {B128, 1024, 1024, 0, true}};
                for (int k = 0; k < subs; ++k) ops.push_back({S, 1024, 1024, 0, true});
                for (int k = 0; k < others; ++k) ops.push_back({B64, 256, 256, 0, true});
                if (run(ops) != MOR_OK || !passes_follow()) return false;
                for (const Launch& l : log_)
                    if (l.second < 0 || l.second > 12) return false;
            }
    return true;
}
// Blocks of any number are accepted beside per-tensor operands; so many that the common launch cannot hold them have their own.
static bool many_blocks() {
    for (int64_t pad = 0; pad <= 4096; pad += 4096)
        for (int64_t rows = 16384; rows <= 16384 * 64; rows *= 4) {
            std::vector<Op> ops{{T, 8192, 4096, pad, false}, {T, 8192, 4096, pad, false}};
            for (int k = 0; k < 8; ++k) ops.push_back({B128, rows, 53248, 0, false});
            if (run(ops) != MOR_OK || !passes_follow() || count("15k_tensor_streamI") != 1 || count("k_team_group") != 1) return false;
            if (run({{T, 4096, 4096, pad, true}, {B128, 1835008, 4096, 0, true}, {B128, 128, 128, 0, true}}) != MOR_OK || !passes_follow()) return false;
        }
    return true;
}
// Tall columns whose scales take a launch of their own stay apart from rows, whether or not columns are proven one by one.
static bool tall_columns() {
    const int R = MOR_GRAN_CHANNEL_ROW, C = MOR_GRAN_CHANNEL_COL;
    for (int scaling : {MOR_SCALE_FP32_AMAX, MOR_SCALE_GAM})
        for (int scope : {MOR_SCOPE_PARTITION, MOR_SCOPE_TENSOR})
            for (int fake = 0; fake < 2; ++fake)
                for (int64_t cols = 128; cols <= 256; cols += 128) {
                    if (run({{C, 65536, cols, 0, false, scaling, scope, fake != 0}, {R, 128, 4096, 0, false, scaling, scope, fake != 0}}) != MOR_OK || !passes_follow()) return false;
                    const int wgs = 4 * (int)cols, limit = fake || scope == MOR_SCOPE_TENSOR ? 512 : 1024;
                    if (count("k_pair_secondI") != (wgs <= limit ? 1 : 0) || count("k_col_scales") != (wgs <= limit ? 0 : 1)) return false;
                }
    return true;
}
// Random mixes of what a batch takes.
static bool mixes() {
    uint64_t state = 1;
    auto draw = [&](int n) { state = state * 6364136223846793005ull + 1442695040888963407ull; return (int)((state >> 33) % (uint64_t)n); };
    for (int round = 0; round < 4000; ++round) {
        std::vector<Op> ops;
        const int n = 1 + draw(round % 4 ? 8 : 40), fakes = draw(4);
        const bool stats = draw(2) != 0;
        for (int k = 0; k < n; ++k) {
            static const int grans[] = {T, T, B128, B128, S, B64, MOR_GRAN_CHANNEL_ROW, MOR_GRAN_CHANNEL_COL};
            Op o{grans[draw(8)], 128ll << draw(6), 128ll << draw(6), draw(3) ? 0 : 128, stats && draw(4) != 0};
            o.scaling = draw(3) ? MOR_SCALE_FP32_AMAX : (draw(2) ? MOR_SCALE_GAM : MOR_SCALE_E8M0);
            if (o.gran != T && !draw(3)) o.scope = MOR_SCOPE_TENSOR;
            o.fake = !fakes && draw(2);
            ops.push_back(o);
        }
        if (run(ops) != MOR_OK || !passes_follow()) return false;
        for (const Launch& l : log_)
            if (l.second < 0 || l.second > 12) return false;
    }
    return true;
}

int main(int, char** argv) {
    void* lib = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
    if (!lib) { fprintf(stderr, "%s\n", dlerror()); return 1; }
    ws_bytes = reinterpret_cast<decltype(ws_bytes)>(dlsym(lib, "mor_batch_workspace_bytes"));
    batch = reinterpret_cast<decltype(batch)>(dlsym(lib, "mor_analyze_quantize_batch"));
    const std::map<std::string, bool (*)()> checks{{"padded_with_blocks", padded_with_blocks}, {"nothing_along", nothing_along}, {"small_alone", small_alone}, {"blocks_that_stay", blocks_that_stay}, {"statistics_fit", statistics_fit}, {"many_blocks", many_blocks}, {"tall_columns", tall_columns}, {"mixes", mixes}};
    printf("%d\n", checks.at(argv[2])() ? 1 : 0);
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    from paper_2512_22804_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    d = tmp_path_factory.mktemp("plans")
    src, exe = d / "plans.cpp", d / "plans"
    src.write_text(SOURCE)
    # (the executable's own definitions come first in the library's symbol search)
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe), "-ldl"], check=True, capture_output=True)
    return lambda check: subprocess.run([str(exe), build.LIB, check], check=True, capture_output=True, text=True, timeout=120).stdout.strip()


@pytest.mark.parametrize("check", ["padded_with_blocks", "nothing_along", "small_alone", "blocks_that_stay", "statistics_fit", "many_blocks", "tall_columns", "mixes"])
def test_plan(driver, check):
    assert driver(check) == "1"
