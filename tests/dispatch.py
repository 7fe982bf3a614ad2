"""Which kernels a call launches, without a GPU: a program of its own whose HIP functions only write down what they are
given, over the library as it is built.  Pointers are made up; nothing on the host reads through them."""
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2310_03675_amd")

PROGRAM = r"""
#include "../../include/hdqt.h"
#include "gemm_lines.hpp"
#include <cxxabi.h>
#include <stdio.h>
#include <string>
#include <map>
#include <string.h>

static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static dim3 g_grid, g_block;
static std::string g_log;

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* stub, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    int rc = 0;
    char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &rc);
    std::string s = rc ? name : plain;
    if (!rc) free(plain);
    const size_t open = s.find("kernel");      // "void hdqt::(anonymous namespace)::name_kernel<...>(...)"
    if (open != std::string::npos) {
        size_t from = s.rfind("::", open);
        from = from == std::string::npos ? 0 : from + 2;
        const size_t to = s.find('(', open);
        s = s.substr(from, to - from);
    }
    names()[stub] = s;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) { g_grid = grid; g_block = block; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream)
{
    *grid = g_grid; *block = g_block; *shared = 0; *stream = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* stub, dim3 grid, dim3 block, void** args, size_t, hipStream_t)
{
    const std::string& name = names()[stub];
    char line[256];
    if (!name.compare(0, 14, "lines_gemm_i4_") || !name.compare(0, 13, "gemm_bytes_ke")) {
        const auto& k = *static_cast<const hdqt::lines::LinesArgs*>(args[0]);
        const unsigned parts = k.tiles / (k.n_rt * k.n_ct);
        snprintf(line, sizeof line, " parts=%u part_codes=%lld slices16=%d", parts, 128ll * k.part_stages, parts > 1 && k.to.partial16);
    } else {
        line[0] = 0;
    }
    g_log += "|" + name + line;
    return (uint64_t)grid.x * block.x >= (1ull << 32) || grid.y > 65535 || grid.z > 65535 ? hipErrorInvalidConfiguration : hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}

int main()
{
    char what[32];
    const hdqt_operand_t op0{4, HDQT_ROUND_NEAREST, 1.0f, 0};
    auto at = [](int k) { return reinterpret_cast<float*>((uintptr_t)(k + 1) << 44); };
    while (scanf("%31s", what) == 1) {
        long long M, K, N, s;
        int b, acc, option;
        if (scanf("%lld %lld %lld %d %d %lld %d", &M, &K, &N, &b, &acc, &s, &option) != 7) return 1;
        hdqt_operand_t op = op0;
        op.b = b;
        hdqt_params_t p{64, acc, s, 0, op, op};
        p.had_block = 1;
        g_log.clear();
        int rc = -99;
        const auto size = [&](int kind) { return hdqt_workspace_size(kind, M, K, N, &p); };
        if (!strcmp(what, "fwd")) rc = hdqt_gemm_fwd(at(0), at(1), at(2), M, K, N, &p, nullptr, at(3), size(HDQT_GEMM_FWD), nullptr);
        if (!strcmp(what, "bwd_weight")) rc = hdqt_gemm_bwd_weight(at(0), at(1), at(2), M, K, N, &p, nullptr, at(3), size(HDQT_GEMM_BWD_WEIGHT), nullptr);
        if (!strcmp(what, "bwd_input")) {      // option: 1 masked, 2 narrowed
            const size_t ws = size(HDQT_GEMM_BWD_INPUT);
            if (option == 1) rc = hdqt_gemm_bwd_input_masked(at(0), at(1), at(4), at(2), M, K, N, &p, nullptr, at(3), ws, nullptr);
            else if (option == 2) rc = hdqt_gemm_bwd_input_bf16(at(0), at(1), (uint16_t*)at(2), M, K, N, &p, nullptr, at(3), ws, nullptr);
            else rc = hdqt_gemm_bwd_input(at(0), at(1), at(2), M, K, N, &p, nullptr, at(3), ws, nullptr);
        }
        if (!strcmp(what, "codes"))            // M x N outputs over K
            rc = hdqt_gemm_codes(at(0), at(1), b, b, at(4), at(5), M, N, K, 1, acc, s, at(2), nullptr, at(3),
                                 hdqt_gemm_codes_workspace_size(M, N, K, s), nullptr);
        if (!strcmp(what, "step"))             // option: 1 without input gradient
            rc = hdqt_layer_step(at(0), at(1), at(2), at(4), option ? nullptr : at(5), at(6), M, K, N, &p, option ? nullptr : &p, &p, at(3),
                                 hdqt_layer_step_workspace_size(M, K, N, &p, option ? nullptr : &p, &p), nullptr);
        // (workspaces of the next larger layer of even sizes: lines as long as hdqt_codes_pitch has them, and no zeros behind)
        const long long M2 = M + M % 2, K2 = K + K % 2, N2 = N + N % 2;
        if (!strcmp(what, "step_even"))
            rc = hdqt_layer_step(at(0), at(1), at(2), at(4), option ? nullptr : at(5), at(6), M, K, N, &p, option ? nullptr : &p, &p, at(3),
                                 hdqt_layer_step_workspace_size(M2, K2, N2, &p, option ? nullptr : &p, &p), nullptr);
        if (!strcmp(what, "layer_fwd_even"))
            rc = hdqt_layer_fwd(at(0), at(1), at(2), M, K, N, &p, &p, at(3), hdqt_layer_saved_size(M, K, &p), at(4),
                                hdqt_layer_fwd_workspace_size(M2, K2, N2, &p, &p), nullptr);
        if (!strcmp(what, "layer_bwd_even"))
            rc = hdqt_layer_bwd(at(0), at(1), at(2), at(3), at(4), M, K, N, &p, &p, at(5),
                                hdqt_layer_bwd_workspace_size(M2, K2, N2, &p, &p), nullptr);
        if (!strcmp(what, "layer_fwd"))
            rc = hdqt_layer_fwd(at(0), at(1), at(2), M, K, N, &p, &p, at(3), hdqt_layer_saved_size(M, K, &p), at(4),
                                hdqt_layer_fwd_workspace_size(M, K, N, &p, &p), nullptr);
        if (!strcmp(what, "layer_bwd")) {      // option: 1 masked
            const size_t ws = hdqt_layer_bwd_workspace_size(M, K, N, &p, &p);
            rc = option ? hdqt_layer_bwd_masked(at(0), at(1), at(2), at(6), at(3), at(4), M, K, N, &p, &p, at(5), ws, nullptr)
                        : hdqt_layer_bwd(at(0), at(1), at(2), at(3), at(4), M, K, N, &p, &p, at(5), ws, nullptr);
        }
        if (!strcmp(what, "conv_bwd")) {       // M images of `option` x `option`, K channels, 3 x 3
            const hdqt_conv_t geo{M, (int32_t)K, option, option, 3, 3};
            rc = hdqt_conv_bwd(at(0), at(1), at(2), &geo, at(3), at(4), N, &p, &p, at(5),
                               hdqt_layer_bwd_workspace_size(M * option * option, 9 * K, N, &p, &p), nullptr);
        }
        printf("%d%s\n", rc, g_log.c_str());
    }
    return 0;
}
"""

_EXE = _FOLDER = None


def _program() -> str:
    global _EXE, _FOLDER
    if _EXE is None:
        _FOLDER = tempfile.TemporaryDirectory(prefix="dispatch")      # (goes with the process)
        folder = _FOLDER.name
        src, exe = os.path.join(folder, "dispatch.hip"), os.path.join(folder, "dispatch")
        with open(src, "w") as f:
            f.write(PROGRAM.replace("../../include", os.path.join(ROOT, "include")))
        hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
        subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-w",
                        "-I", os.path.join(PACKAGE, "csrc"), "-c", src, "-o", exe + ".o"], check=True)
        # (-rdynamic: the library's HIP calls find the program's functions before HIP's own)
        subprocess.run(["g++", "-rdynamic", exe + ".o", os.path.join(PACKAGE, "libhdqt.so"), "-Wl,--allow-shlib-undefined",
                        f"-Wl,-rpath,{PACKAGE}", "-o", exe], check=True)
        _EXE = exe
    return _EXE


def dispatch(calls):
    """calls: (entry point, M, K, N, b, acc, s, option) each; what each returns, and the kernels it launches."""
    text = "".join(" ".join(map(str, c)) + "\n" for c in calls)
    out = subprocess.run([_program()], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(out) == len(calls)
    return [(int(line.split("|")[0]), line.split("|")[1:]) for line in out]
