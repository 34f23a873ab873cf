// Runs the host side of the actor step, as built in libpcm.so, on a HIP runtime of its own that launches nothing: the
// functions below take the place of the runtime's, so no GPU is needed or touched.  Every launch of a matrix product, of
// a sum of parts and, on the fp32 path, of everything else is looked at as the library issues it: each matrix that it reads or
// writes has to lie inside one of the buffers that the call was given, apart from what the launch writes; the workspace is as
// long as the library's own query says, or as short as a call accepts.  A kernel that is neither known here nor listed as left
// out is a failure.
//
//   host_path bounds   sweeps sizes and options and checks every launch
//   host_path errors   lets each launch of a call fail in turn: the call has to return PCM_EHIP
//   host_path least    the fp32 calls again, with the shortest workspace that they accept
#include <cxxabi.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "actor_f32.h"
#include "epilogues_f32.h"
#include "gemm_bf16.h"
#include "gemm_direct.h"
#include "pcm.h"

using namespace pcm;

namespace {

struct Region {
    const char* what;
    uintptr_t begin, end;
};
std::vector<Region> regions;                      // what the call may touch
std::map<const void*, std::string>& kernel_names() {   // by host stub; the library registers its kernels before main
    static std::map<const void*, std::string> names;
    return names;
}
std::string call;                                 // the call under way
int failures = 0, launches = 0, products = 0, sums = 0;
int fail_at = -1;                                 // the launch that fails, or -1
bool check_bounds = false;
hipError_t last_error = hipSuccess;

template <class T>
T* buffer(const char* what, size_t count) {
    const uintptr_t begin = regions.empty() ? (uintptr_t)1 << 40 : (regions.back().end + (1u << 20)) / 4096 * 4096;
    regions.push_back(Region{what, begin, begin + count * sizeof(T)});
    return reinterpret_cast<T*>(begin);
}
// What a launch touches: two matrices of which one is written, the epilogue's or the launch's result, may not share memory, unless they
// are the same one (in place).
struct Span {
    const char* what;
    uintptr_t begin, end;
    bool written;
};
std::vector<Span> spans;
bool writing = false;
void check_overlaps(const char* kernel) {
    for (size_t a = 0; a < spans.size(); ++a)
        for (size_t b = 0; b < a; ++b) {
            const Span &p = spans[a], &q = spans[b];
            if (!(p.written || q.written) || p.begin == q.begin || p.end <= q.begin || q.end <= p.begin) continue;
            if (++failures <= 20) printf("%s\n  %s: %s and %s share memory\n", call.c_str(), kernel, p.what, q.what);
        }
    spans.clear();
}
// `rows` rows of `columns` values, ld apart
void touches(const char* kernel, const char* what, const void* p, int64_t rows, int64_t columns, int64_t ld, size_t size) {
    if (rows <= 0) return;
    const uintptr_t begin = (uintptr_t)p, end = begin + (uintptr_t)((rows - 1) * ld + columns) * size;
    spans.push_back(Span{what, begin, end, writing});
    for (const Region& r : regions)
        if (begin >= r.begin && end <= r.end) return;
    if (++failures > 20) return;
    const char* in = "no buffer";
    long long beyond = 0;
    for (const Region& r : regions)
        if (begin >= r.begin && begin < r.end) { in = r.what; beyond = (long long)(end - r.end); }
    printf("%s\n  %s: %s [%lld x %lld] starts in %s and ends %lld bytes beyond it\n", call.c_str(), kernel, what, (long long)rows,
           (long long)columns, in, beyond);
}

// What the epilogues write; what they read of matrices is what they write, or as large.
void writes(const char* k, const GemmProblem& p, const EpiStoreF32& e) {
    for (int s = 0; s < p.splits; ++s) touches(k, "fp32 result", e.C + s * e.split_stride, p.M, p.N, e.ldc, 4);
}
void writes(const char* k, const GemmProblem& p, const EpiStoreBf16& e) {
    touches(k, "bf16 result", e.C, p.M < e.row_limit ? p.M : e.row_limit, p.N, e.ldc, 2);
}
void writes(const char* k, const GemmProblem& p, const EpiStoreBf16Split& e) {
    for (const bf16* q : {e.hi, e.lo}) touches(k, "bf16 pair", q, p.M < e.row_limit ? p.M : e.row_limit, p.N, e.ldc, 2);
}
void writes(const char* k, const GemmProblem& p, const EpiScatterBf16& e) { touches(k, "list", e.row_idx, 1, p.M, p.M, 4); }
template <bool kFactors, bool kLow>
void writes(const char* k, const GemmProblem& p, const EpiSwigluForward<kFactors, kLow>& e) {
    touches(k, "a", e.a, p.M, p.N / 2, e.ld, 2);
    if (kFactors) for (const bf16* q : {e.fu, e.fv}) touches(k, "factor", q, p.M, p.N / 2, e.ld, 2);
    if (kLow) touches(k, "a_lo", e.a_lo, p.M, p.N / 2, e.ld, 2);
}
template <bool kIndexed>
void writes(const char* k, const GemmProblem& p, const EpiSwigluBackward<kIndexed>& e) {
    for (const bf16* q : {e.fu, e.fv}) touches(k, "factor", q, p.M, p.N, e.ld, 2);
    if (kIndexed) for (const bf16* q : {e.du, e.dv}) touches(k, "du, dv", q, p.M, p.N, e.ld, 2);
    if (kIndexed) touches(k, "list", e.row_idx, 1, p.M, p.M, 4);
}
template <int kLayA, int kLayB>
void reads(const char* k, const GemmProblem& p) {
    const bf16* const operand[2][2] = {{p.A, p.A2}, {p.B, p.B2}};
    for (int segment = 0; segment < (p.K2 > 0 ? 2 : 1); ++segment) {
        const int K = segment ? p.K2 : p.K1;
        if (kLayA == kRowsByK) touches(k, "A", operand[0][segment], p.M, K, p.lda, 2);
        else touches(k, "A", operand[0][segment], K, p.M, p.lda, 2);
        if (kLayB == kRowsByK) touches(k, "B", operand[1][segment], p.N, K, p.ldb, 2);
        else touches(k, "B", operand[1][segment], K, p.N, p.ldb, 2);
    }
}
template <int kLayA, int kLayB, class Epilogue>
void look(const char* k, const GemmProblem& p, const Epilogue& e) {
    reads<kLayA, kLayB>(k, p);
    writing = true;
    writes(k, p, e);
    writing = false;
    ++products;
}
template <int kLayA, int kLayB, class Epilogue>
void look_at_job(const char* k, const void* arg) {
    const auto& j = *static_cast<const GemmJob<kLayA, kLayB, Epilogue>*>(arg);
    look<kLayA, kLayB>(k, j.p, j.epi);
}
template <int kLayA, int kLayB, class Epilogue>
void look_at_pair(const char* k, const void* arg) {
    auto j = *static_cast<const GemmPairJob<kLayA, kLayB, Epilogue>*>(arg);
    for (int q = 0; q < 2; ++q) {
        j.p.B = j.p.B2 = j.B[q];
        look<kLayA, kLayB>(k, j.p, j.epi[q]);
    }
}

void unknown(const std::string& what) {
    if (++failures <= 20) printf("%s\n  a launch that this program does not know: %s\n", call.c_str(), what.c_str());
}
void require(bool ok, const char* kernel, const char* what) {
    if (!ok && ++failures <= 20) printf("%s\n  %s: %s\n", call.c_str(), kernel, what);
}

// ---- fp32: operands in blocks of 128 rows x 32 columns, whole blocks; columns up to `columns` are used
int64_t padded(int64_t n) { return (n + kThirdsUnit - 1) / kThirdsUnit * kThirdsUnit; }
void touches_blocks(const char* k, const char* what, const void* p, int64_t rows, int64_t columns, int64_t ld, size_t size) {
    require(columns <= ld && ld % kThirdsUnit == 0, k, "columns beyond the blocks");
    touches(k, what, p, padded(rows), ld, ld, size);
}
void touches(const char* k, const char* what, const FloatBlocks& m, int64_t rows, int64_t columns) { touches_blocks(k, what, m.p, rows, columns, m.ld, 4); }
void touches(const char* k, const char* what, const Thirds& m, int64_t rows, int64_t columns) { touches_blocks(k, what, m.p, rows, columns, m.ld, 6); }

void writes(const char* k, const FloatsProblem& p, const EpiGateUp& e) {
    if (e.uv != nullptr) touches(k, "u and v", e.uv, p.M, 2 * e.a.ld, 2 * e.a.ld, 4);
    touches(k, "a", e.a, p.M, p.N / 2);
    if (e.a3.p != nullptr) touches(k, "a as thirds", e.a3, p.M, p.N / 2);
}
void writes(const char* k, const FloatsProblem& p, const EpiOperand& e) {
    touches(k, "result", e.C, p.M, p.N);
    if (e.C3.p != nullptr) touches(k, "result as thirds", e.C3, p.M, p.N);
}
void writes(const char* k, const FloatsProblem& p, const EpiRows& e) { touches(k, "rows", e.C, p.M, p.N, e.ldc, 4); }
template <class Epilogue>
void look_at_floats(const char* k, void** args) {
    const FloatsProblem& p = *static_cast<FloatsProblem*>(args[0]);
    require(p.M % 64 == 0 && p.N % 64 == 0 && p.K % 32 == 0 && p.K > 0, k, "sizes that are no multiples of the tile");
    touches(k, "A", FloatBlocks{const_cast<float*>(p.A), p.lda}, p.M, p.K);
    touches(k, "B", FloatBlocks{const_cast<float*>(p.B), p.ldb}, p.N, p.K);
    writing = true;
    writes(k, p, *static_cast<Epilogue*>(args[1]));
    writing = false;
    ++products;
}

void writes(const char* k, const GemmProblem&, const EpiThirds& e) { touches(k, "thirds", e.C, e.rows, e.C.ld); }
void writes(const char* k, const GemmProblem& p, const EpiFloats& e) {
    for (int s = 0; s < p.splits; ++s) touches(k, "fp32 result", e.C + s * e.split_stride, e.M, e.N, e.ldc, 4);
    require(e.M <= p.M && e.N <= p.N, k, "a result wider than the product");
}
void writes(const char* k, const GemmProblem& p, const EpiFloatsPair& e) {
    for (int s = 0; s < p.splits; ++s)
        for (float* C : e.C) touches(k, "one of two fp32 results", C + s * e.split_stride, e.M, e.N, e.N, 4);
    require(e.M <= p.M && 2 * e.N <= p.N, k, "a result wider than the product");
}
void writes(const char* k, const GemmProblem& p, const EpiGateUpBackward& e) {
    touches(k, "u and v", e.uv, p.M, e.duv.ld, e.duv.ld, 4);
    touches(k, "du and dv", e.duv, p.M, e.duv.ld);
    require(e.duv.ld <= 2 * (int64_t)p.N, k, "du and dv wider than the product");
}
template <int kLayA, int kLayB, class Epilogue>
void look_at_thirds(const char* k, const void* arg) {
    const auto& j = *static_cast<const ThirdsProduct<kLayA, kLayB, Epilogue>*>(arg);
    GemmProblem p = j.p;
    require(p.M % kThirdsUnit == 0 && p.N % kThirdsUnit == 0 && p.K1 % kTileK == 0 && p.K1 > 0, k, "sizes that are no multiples of the tile");
    require(p.splits >= 1 && p.splits <= 64 && j.first % 8 == 0, k, "parts");
    const Thirds A{const_cast<bf16*>(p.A), p.lda}, B{const_cast<bf16*>(p.B), p.ldb};
    touches(k, "A", A, kLayA == kRowsByK ? p.M : p.K1, kLayA == kRowsByK ? p.K1 : p.M);
    touches(k, "B", B, kLayB == kRowsByK ? p.N : p.K1, kLayB == kRowsByK ? p.K1 : p.N);
    writing = true;
    writes(k, p, j.epi);
    writing = false;
    ++products;
}

// ---- fp32, direct route
template <int kLayA, int kLayB>
void reads_direct(const char* k, const F32Problem& p, int second) {
    const float* const operand[2][2] = {{p.A, p.A2}, {p.B, p.B2}};
    for (int q = 0; q < (second == kNone ? 1 : 2); ++q) {
        const float* const A = operand[0][second == kSum ? q : 0];
        if (kLayA == kRowsByK) touches(k, "A", A, p.M, p.K, p.lda, 4);
        else touches(k, "A", A, p.K, p.M, p.lda, 4);
        if (kLayB == kRowsByK) touches(k, "B", operand[1][q], p.N, p.K, p.ldb, 4);
        else touches(k, "B", operand[1][q], p.K, p.N, p.ldb, 4);
    }
}
void writes(const char* k, const F32Problem& p, int second, int slices, const F32Store& e) {
    for (int z = 0; z < slices; ++z)
        for (float* C : {e.C, second == kPair ? e.C2 : e.C}) touches(k, "result", C + z * e.split_stride, p.M, p.N, e.ldc, 4);
}
void writes(const char* k, const F32Problem& p, int, int, const F32SwigluForward& e) {
    for (float* C : {e.u, e.v, e.a}) touches(k, "u, v or a", C, p.M, p.N, p.N, 4);
}
void writes(const char* k, const F32Problem& p, int, int, const F32SwigluBackward& e) {
    for (float* C : {e.u, e.v}) touches(k, "u or v", C, p.M, p.N, p.N, 4);
}
template <class Epilogue>
void look_at_direct(const char* k, int lay_a, int lay_b, int second, int slices, void** args) {
    const F32Problem& p = *static_cast<F32Problem*>(args[0]);
    if (lay_a == kRowsByK && lay_b == kRowsByK) reads_direct<kRowsByK, kRowsByK>(k, p, second);
    else if (lay_a == kRowsByK) reads_direct<kRowsByK, kKByRows>(k, p, second);
    else reads_direct<kKByRows, kKByRows>(k, p, second);
    require((int64_t)slices * p.k_per_split >= p.K || second == kSum, k, "slices that leave out some of the reduction");
    writing = true;
    writes(k, p, second, slices, *static_cast<Epilogue*>(args[1]));
    writing = false;
    ++products;
}

// ---- fp32, the other launches
template <class Vec>
void reads(const char* k, const GatherArgs<Vec>& g) {
    const int64_t all = (int64_t)g.T * g.N * g.A;
    touches(k, "hidden", g.hidden, all, g.vec_per_row, g.vec_per_row, sizeof(Vec));
    touches(k, "tokens", g.tokens, 1, all, all, 1);
    touches(k, "logp_old", g.logp_old, 1, all, all, 4);
    touches(k, "adv", g.adv, 1, g.T, g.T, 4);
    touches(k, "row tokens", g.meta.token, 1, g.rows_pad, g.rows_pad, 1);
    for (const float* q : {g.meta.logp_old, g.meta.adv}) touches(k, "row metadata", q, 1, g.rows_pad, g.rows_pad, 4);
}
void look_at_prepare(const char* k, const PrepareF32& p) {
    const GatherArgs<float>& g = p.gather;
    const int64_t d = g.vec_per_row;
    reads(k, g);
    require(g.rows_pad % 256 == 0 && p.X.ld == padded(d), k, "X");
    writing = true;
    touches(k, "X", p.X, g.rows_pad, p.X.ld);
    if (p.X3.p != nullptr) touches(k, "X as thirds", p.X3, g.rows_pad, p.X.ld);
    if (p.dX != nullptr) touches(k, "dX", p.dX, (int64_t)g.max_chunks * g.A, d, d, 4);
    for (int q = 0; q < p.weights.n; ++q) {
        const WeightJob& j = p.weights.job[q];
        writing = false;
        touches(k, "a weight", j.src, j.R, j.C, j.C, 4);
        writing = true;
        const int64_t columns = padded(j.C) * (j.mode == kPackNone ? 1 : 2), rows = padded(j.R);
        if (j.transposed) touches(k, "a weight as floats", j.to, columns, rows);
        else if (j.to.p != nullptr) touches(k, "a weight as floats", j.to, rows, columns);
        else touches(k, "a weight as thirds", j.to3, rows, columns);
    }
    writing = false;
}
void look_at_loss(const char* k, const LossArgs& p) {
    writing = true;
    touches(k, "z", p.z, p.rows, p.ld, p.ld, 4);
    if (p.opt.chunk_ratio && (p.dz.p != nullptr || p.in_place)) {
        const int64_t live = (int64_t)p.max_chunks * p.A;
        touches(k, "extra", p.extra, p.rows < live ? p.rows : live, p.V, p.V, 4);
    }
    if (p.dz.p != nullptr) touches(k, "dz", p.dz, p.rows, p.ld);
    touches(k, "row tokens", p.meta.token, 1, p.rows, p.rows, 1);
    for (const float* q : {p.meta.logp_old, p.meta.adv, p.out.dlogp, p.out.entropy, p.out.term, p.out.ratio})
        touches(k, "a value per row", q, 1, p.rows, p.rows, 4);
    touches(k, "clip flags", p.out.clipped, 1, p.rows, p.rows, 1);
    writing = false;
}

// The parts of a template argument list "A<..>, B, ..": split at the commas of the outermost level.
std::vector<std::string> arguments(const std::string& text, size_t open) {
    std::vector<std::string> parts(1);
    int depth = 0;
    for (size_t i = open + 1; i < text.size(); ++i) {
        const char c = text[i];
        if (c == '<') ++depth;
        if (c == '>' && depth-- == 0) break;
        if (c == ',' && depth == 0) parts.emplace_back();
        else if (c != ' ') parts.back() += c;
    }
    return parts;
}
using Look = void (*)(const char*, const void*);
// Job types by name, as the demangled kernel names write them without blanks.
template <int kLayA, int kLayB, class Epilogue>
void add_job(std::map<std::string, Look>& jobs, const char* epilogue) {
    const std::string layouts = std::to_string(kLayA) + "," + std::to_string(kLayB) + ",";
    jobs["pcm::GemmJob<" + layouts + epilogue + ">"] = look_at_job<kLayA, kLayB, Epilogue>;
}
template <class Epilogue>
void add_jobs(std::map<std::string, Look>& jobs, const char* epilogue) {
    add_job<0, 0, Epilogue>(jobs, epilogue);
    add_job<0, 1, Epilogue>(jobs, epilogue);
    add_job<1, 1, Epilogue>(jobs, epilogue);
}
const std::map<std::string, Look>& known_jobs() {
    static std::map<std::string, Look> jobs;
    if (jobs.empty()) {
        add_jobs<EpiStoreF32>(jobs, "pcm::EpiStoreF32");
        add_jobs<EpiStoreBf16>(jobs, "pcm::EpiStoreBf16");
        add_jobs<EpiStoreBf16Split>(jobs, "pcm::EpiStoreBf16Split");
        add_jobs<EpiScatterBf16>(jobs, "pcm::EpiScatterBf16");
        add_jobs<EpiSwigluForward<false, false>>(jobs, "pcm::EpiSwigluForward<false,false>");
        add_jobs<EpiSwigluForward<false, true>>(jobs, "pcm::EpiSwigluForward<false,true>");
        add_jobs<EpiSwigluForward<true, false>>(jobs, "pcm::EpiSwigluForward<true,false>");
        add_jobs<EpiSwigluForward<true, true>>(jobs, "pcm::EpiSwigluForward<true,true>");
        add_jobs<EpiSwigluBackward<false>>(jobs, "pcm::EpiSwigluBackward<false>");
        add_jobs<EpiSwigluBackward<true>>(jobs, "pcm::EpiSwigluBackward<true>");
        jobs["pcm::GemmPairJob<1,1,pcm::EpiStoreF32>"] = look_at_pair<1, 1, EpiStoreF32>;
        jobs["pcm::ThirdsProduct<0,0,pcm::EpiThirds>"] = look_at_thirds<0, 0, EpiThirds>;
        jobs["pcm::ThirdsProduct<0,0,pcm::EpiFloats>"] = look_at_thirds<0, 0, EpiFloats>;
        jobs["pcm::ThirdsProduct<1,1,pcm::EpiFloats>"] = look_at_thirds<1, 1, EpiFloats>;
        jobs["pcm::ThirdsProduct<0,0,pcm::EpiFloatsInChains>"] = look_at_thirds<0, 0, EpiFloatsInChains>;
        jobs["pcm::ThirdsProduct<1,1,pcm::EpiFloatsInChains>"] = look_at_thirds<1, 1, EpiFloatsInChains>;
        jobs["pcm::ThirdsProduct<1,1,pcm::EpiFloatsPair>"] = look_at_thirds<1, 1, EpiFloatsPair>;
        jobs["pcm::ThirdsProduct<0,0,pcm::EpiGateUpBackward>"] = look_at_thirds<0, 0, EpiGateUpBackward>;
        jobs["pcm::ThirdsProduct<0,1,pcm::EpiGateUpBackward>"] = look_at_thirds<0, 1, EpiGateUpBackward>;
    }
    return jobs;
}
// A product by itself has the arguments (GemmProblem, epilogue); a job holds the two side by side.
void look_at_product(const char* k, const std::string& layouts_and_epilogue, void** args);

void look_at_launch(const std::string& name, void** args, dim3 grid) {
    size_t at = name.find("gemm_f32<");
    if (at != std::string::npos) {
        const auto parts = arguments(name, at + strlen("gemm_f32<") - 1);
        for (size_t q = 0; q < parts.size(); ++q) {
            const auto job = known_jobs().find(parts[q]);
            if (job == known_jobs().end()) unknown(parts[q]);
            else job->second(parts[q].c_str(), args[q]);
        }
        return;
    }
    at = name.find("gemm_floats<");
    if (at != std::string::npos) {
        const std::string epilogue = arguments(name, at + strlen("gemm_floats<") - 1)[2];
        if (epilogue == "pcm::EpiGateUp") look_at_floats<EpiGateUp>("gemm_floats, gate and up", args);
        else if (epilogue == "pcm::EpiOperand") look_at_floats<EpiOperand>("gemm_floats to an operand", args);
        else if (epilogue == "pcm::EpiRows") look_at_floats<EpiRows>("gemm_floats to rows", args);
        else unknown(name);
        return;
    }
    at = name.find("gemm_direct<");
    if (at != std::string::npos) {                      // tile, tile, layout, layout, second product, vectors, epilogue
        const auto parts = arguments(name, at + strlen("gemm_direct<") - 1);
        const int lay_a = atoi(parts[2].c_str()), lay_b = atoi(parts[3].c_str()), second = atoi(parts[4].c_str()), slices = (int)grid.z;
        if (parts[6] == "pcm::F32Store") look_at_direct<F32Store>("gemm_direct", lay_a, lay_b, second, slices, args);
        else if (parts[6] == "pcm::F32SwigluForward") look_at_direct<F32SwigluForward>("gemm_direct, gate and up", lay_a, lay_b, second, slices, args);
        else if (parts[6] == "pcm::F32SwigluBackward") look_at_direct<F32SwigluBackward>("gemm_direct, da", lay_a, lay_b, second, slices, args);
        else unknown(name);
        return;
    }
    at = name.find("gemm_group<");
    if (at != std::string::npos) {
        const auto parts = arguments(name, at + strlen("gemm_group<") - 1);
        for (size_t q = 2; q < parts.size(); ++q) {
            const auto job = known_jobs().find(parts[q]);
            if (job == known_jobs().end()) unknown(parts[q]);
            else job->second(parts[q].c_str(), args[q - 2]);
        }
        return;
    }
    at = name.find("gemm_bf16<");
    if (at != std::string::npos) {
        const auto parts = arguments(name, at + strlen("gemm_bf16<") - 1);      // epilogue, layout, layout, tile, ring
        look_at_product(parts[0].c_str(), parts[1] + "," + parts[2] + "," + parts[0], args);
        return;
    }
    if (name.find("sum_parts_bf16") != std::string::npos) {
        const int n_parts = *static_cast<int*>(args[1]);
        const size_t n = *static_cast<size_t*>(args[2]);
        touches("sum_parts_bf16", "parts", *static_cast<void**>(args[0]), n_parts, (int64_t)n, (int64_t)n, 4);
        touches("sum_parts_bf16", "result", *static_cast<void**>(args[3]), 1, (int64_t)n, (int64_t)n, 2);
        ++sums;
        return;
    }
    const auto is = [&](const char* kernel) { return name.find(std::string("::") + kernel + "(") != std::string::npos; };
    if (is("sum_parts_thirds")) {
        const int n_parts = *static_cast<int*>(args[1]);
        const int64_t n = (int64_t)*static_cast<size_t*>(args[2]);
        const Thirds C = *static_cast<Thirds*>(args[3]);
        touches("sum_parts_thirds", "parts", *static_cast<void**>(args[0]), n_parts, n, n, 4);
        require(n % C.ld == 0, "sum_parts_thirds", "rows in part");
        writing = true;
        touches("sum_parts_thirds", "result", C, n / C.ld, C.ld);
        writing = false;
        ++sums;
        return;
    }
    if (is("prepare_step_f32")) return look_at_prepare("prepare_step_f32", *static_cast<PrepareF32*>(args[0]));
    if (name.find("::loss_rows<") != std::string::npos) return look_at_loss("loss_rows", *static_cast<LossArgs*>(args[0]));
    if (is("scale_rows")) {                             // z, extra or null, V, coef, n_kept, max_chunks, A, dz
        const int64_t V = *static_cast<int*>(args[2]), rows = (int64_t)*static_cast<int*>(args[5]) * *static_cast<int*>(args[6]);
        const Thirds dz = *static_cast<Thirds*>(args[7]);
        touches("scale_rows", "z", *static_cast<float**>(args[0]), rows, dz.ld, dz.ld, 4);
        if (float* const extra = *static_cast<float**>(args[1])) touches("scale_rows", "extra", extra, rows, V, V, 4);
        touches("scale_rows", "coefficients", *static_cast<float**>(args[3]), 1, rows, rows, 4);
        writing = true;
        touches("scale_rows", "dz", dz, (rows + 255) / 256 * 256, dz.ld);
        writing = false;
        return;
    }
    if (is("scale_rows_f32")) {                         // dz, extra or null, coef, n_kept, max_chunks, A, rows, V
        const int64_t rows = *static_cast<int64_t*>(args[6]), V = *static_cast<int*>(args[7]);
        touches("scale_rows_f32", "dz", *static_cast<float**>(args[0]), rows, V, V, 4);
        if (float* const extra = *static_cast<float**>(args[1])) touches("scale_rows_f32", "extra", extra, rows, V, V, 4);
        touches("scale_rows_f32", "coefficients", *static_cast<float**>(args[2]), 1, rows, rows, 4);
        return;
    }
    at = name.find("prepare_step<");
    if (at != std::string::npos) {
        const std::string vec = arguments(name, at + strlen("prepare_step<") - 1)[0];
        const auto look = [&](auto unit) {
            const auto& g = *static_cast<GatherArgs<decltype(unit)>*>(args[0]);
            reads("prepare_step", g);
            writing = true;
            touches("prepare_step", "X", g.X, g.rows_pad, g.vec_per_row, g.vec_per_row, sizeof unit);
            writing = false;
        };
        if (vec.find("4") != std::string::npos) look(uint4{});
        else if (vec == "unsignedint") look(uint32_t{});
        else if (vec == "unsignedshort") look(uint16_t{});
        else unknown(name);
        return;
    }
    if (name.find("finish_step") != std::string::npos) {
        const PartsSums& s = *static_cast<PartsSums*>(args[0]);
        for (int q = 0; q < s.n; ++q) {
            touches("finish_step", "parts", s.job[q].parts, s.job[q].n_parts, (int64_t)s.job[q].n, (int64_t)s.job[q].stride, 4);
            writing = true;
            touches("finish_step", "result", s.job[q].out, 1, (int64_t)s.job[q].n, (int64_t)s.job[q].n, 4);
            writing = false;
            if (s.job[q].sumsq) touches("finish_step", "squares", s.job[q].sumsq, 1, s.job[q].blocks, s.job[q].blocks, 8);
            ++sums;
        }
        return;
    }
    // left out: a value or two per row, and the bf16 path's copies of listed rows and of weights
    for (const char* kernel : {"finish_loss", "chunk_ratio_rows", "list_live_rows", "loss_rows_bf16", "scale_rows_bf16", "transpose_weights",
                               "sum_of_squares"})
        if (name.find(kernel) != std::string::npos) return;
    unknown(name);
}
template <class Epilogue, int kLayA, int kLayB>
void look_at_args(const char* k, void** args) {
    look<kLayA, kLayB>(k, *static_cast<GemmProblem*>(args[0]), *static_cast<Epilogue*>(args[1]));
}
template <class Epilogue>
bool try_epilogue(const char* k, const std::string& want, const char* name, void** args) {
    if (want == std::string("0,0,") + name) return look_at_args<Epilogue, 0, 0>(k, args), true;
    if (want == std::string("0,1,") + name) return look_at_args<Epilogue, 0, 1>(k, args), true;
    if (want == std::string("1,1,") + name) return look_at_args<Epilogue, 1, 1>(k, args), true;
    return false;
}
void look_at_product(const char* k, const std::string& w, void** args) {
    if (try_epilogue<EpiStoreF32>(k, w, "pcm::EpiStoreF32", args) || try_epilogue<EpiStoreBf16>(k, w, "pcm::EpiStoreBf16", args) ||
        try_epilogue<EpiStoreBf16Split>(k, w, "pcm::EpiStoreBf16Split", args) ||
        try_epilogue<EpiScatterBf16>(k, w, "pcm::EpiScatterBf16", args) ||
        try_epilogue<EpiSwigluForward<false, false>>(k, w, "pcm::EpiSwigluForward<false,false>", args) ||
        try_epilogue<EpiSwigluForward<false, true>>(k, w, "pcm::EpiSwigluForward<false,true>", args) ||
        try_epilogue<EpiSwigluForward<true, false>>(k, w, "pcm::EpiSwigluForward<true,false>", args) ||
        try_epilogue<EpiSwigluForward<true, true>>(k, w, "pcm::EpiSwigluForward<true,true>", args) ||
        try_epilogue<EpiSwigluBackward<false>>(k, w, "pcm::EpiSwigluBackward<false>", args) ||
        try_epilogue<EpiSwigluBackward<true>>(k, w, "pcm::EpiSwigluBackward<true>", args))
        return;
    unknown(w);
}

}  // namespace

// ---- the runtime -------------------------------------------------------------------------------
extern "C" {
struct CallConfiguration { dim3 grid, block; size_t shared; hipStream_t stream; };
static CallConfiguration configuration;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
    configuration = CallConfiguration{grid, block, shared, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
    *grid = configuration.grid; *block = configuration.block; *shared = configuration.shared; *stream = configuration.stream;
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* stub, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) {
    int status = 0;
    char* const text = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    kernel_names()[stub] = text ? text : name;
    free(text);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t hipLaunchKernel(const void* stub, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
    const bool fails = launches++ == fail_at;
    if (fails) return last_error = hipErrorLaunchFailure;
    if (check_bounds) {
        if (grid.x == 0 || grid.y == 0 || grid.z == 0 || grid.y > 65535 || grid.z > 65535 || block.x * block.y * block.z > 1024) unknown("an empty or too large grid");
        spans.clear();
        look_at_launch(kernel_names()[stub], args, grid);
        check_overlaps(kernel_names()[stub].substr(0, 200).c_str());
    }
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
hipError_t hipGetDevice(int* device) { *device = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidSymbol; }
hipError_t hipEventCreate(hipEvent_t*) { return hipErrorInvalidValue; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorInvalidValue; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorInvalidValue; }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipErrorInvalidValue; }
}

namespace {

struct Step {
    int dtype, chunks, A, d, ff, V;
    bool weights, dX, composed, chunk_ratio, sumsq, packed, dense;
    float entropy;
    int panel_rows;
};
size_t query = 0;                                 // what the last call's query said
int run(const Step& c, size_t workspace_bytes = 0) {
    char text[256];
    snprintf(text, sizeof text, "dtype %d, %d chunks of %d rows, %d -> %d -> %d, weights %d dX %d composed %d chunk ratio %d squares %d "
             "packed %d dense %d entropy %g panels %d", c.dtype, c.chunks, c.A, c.d, c.ff, c.V, c.weights, c.dX, c.composed, c.chunk_ratio,
             c.sumsq, c.packed, c.dense, c.entropy, c.panel_rows);
    call = text;
    regions.clear();
    const size_t d = c.d, ff = c.ff, V = c.V, rows = (size_t)c.chunks * c.A, size = c.dtype == PCM_BF16 ? 2 : 4;
    pcm_loss_options o{};
    o.eps_low = o.eps_high = 0.2f;
    o.loss_scale = 1.f;
    o.entropy_coef = c.entropy;
    o.ratio_level = c.chunk_ratio ? PCM_RATIO_CHUNK : PCM_RATIO_TOKEN;
    o.head_evaluation = c.composed ? PCM_HEAD_COMPOSED : PCM_HEAD_AS_WRITTEN;
    o.panel_rows = c.panel_rows;
    o.dense_backward = c.dense;
    if (c.packed) o.packed_weights = buffer<char>("packed weights", pcm_packed_head_bytes(c.d, c.ff, c.V));
    if (c.sumsq) o.grad_sumsq_out = buffer<double>("sum of squares", 1);
    const char* const hidden = buffer<char>("hidden", rows * d * size);
    const uint8_t* const tokens = buffer<uint8_t>("tokens", rows);
    const float* const logp_old = buffer<float>("logp_old", rows);
    const float* const adv = buffer<float>("adv", c.chunks);
    const int32_t* const kept = buffer<int32_t>("kept_idx", c.chunks);
    const int32_t* const n_kept = buffer<int32_t>("n_kept", 1);
    const char *const Wg = buffer<char>("Wg", d * ff * size), *const Wu = buffer<char>("Wu", d * ff * size);
    const char *const Wd = buffer<char>("Wd", ff * d * size), *const Wo = buffer<char>("Wo", d * V * size);
    float* const loss = buffer<float>("loss", 1);
    float *dW[4] = {};
    if (c.weights) {
        const size_t n[4] = {d * ff, d * ff, ff * d, d * V};
        for (int q = 0; q < 4; ++q) dW[q] = buffer<float>("a weight gradient", n[q]);
    }
    char* const dX = c.dX ? buffer<char>("dX", rows * d * size) : nullptr;
    size_t bytes = grpo_masked_actor_step_ex_workspace_bytes(c.chunks, c.A, c.d, c.ff, c.V, c.dtype, c.weights || c.dX, &o);
    if (bytes == 0) { unknown("the workspace query refuses the shape"); return PCM_EINVAL; }
    query = bytes;
    if (workspace_bytes != 0) bytes = workspace_bytes;
    char* const ws = buffer<char>("the workspace", bytes);
    launches = 0;
    last_error = hipSuccess;
    return grpo_masked_actor_step_ex(hidden, tokens, logp_old, adv, kept, n_kept, c.chunks, c.chunks, 1, c.A, c.d, c.ff, c.V, c.dtype, Wg, Wu,
                                     Wd, Wo, &o, loss, nullptr, dW[0], dW[1], dW[2], dW[3], dX, nullptr, ws, bytes, nullptr);
}
void expect(int rc, int want) {
    if (rc != want && ++failures <= 20) printf("%s\n  returned %d, not %d\n", call.c_str(), rc, want);
}

// f over the bf16 calls of one size
template <class F>
void bf16_calls(int chunks, int A, int d, int ff, int panel_rows, F f) {
    Step s{PCM_BF16, chunks, A, d, ff, 256, false, false, false, false, false, false, false, 0.f, panel_rows};
    for (int composed = 0; composed < 2; ++composed)
        for (int grads = 0; grads < 4; ++grads)
            for (int option = 0; option < 5; ++option) {
                Step c = s;
                c.composed = composed;
                c.weights = grads & 1;
                c.dX = grads & 2;
                c.packed = option == 1 && !composed;
                c.chunk_ratio = option == 2 && !composed;
                c.sumsq = (option == 1 || option == 4) && c.weights && !composed;
                c.dense = option == 3;
                c.entropy = option == 4 ? 1e-3f : 0.f;
                f(c);
            }
}
// f over the fp32 calls
template <class F>
void f32_calls(F f) {
    auto calls = [&](int chunks, int A, int d, int ff, int V) {
        for (int q = 0; q < 16; ++q)
            f(Step{PCM_F32, chunks, A, d, ff, V, (q & 1) != 0, (q & 2) != 0, (q & 4) != 0, (q & 8) != 0, false, false, false, q % 3 == 0 ? 1e-3f : 0.f, 0});
    };
    for (int d : {1, 33, 64, 65, 128, 129, 256, 1024})
        for (int ff : {1, 64, 65, 127, 300, 2816})
            for (int V : {1, 17, 256, 1024})
                for (int chunks : {1, 9, 46, 500}) calls(chunks, 56, d, ff, V);
    for (int chunks : {1, 2, 64, 65, 256, 257, 300}) calls(chunks, 1, 4096, 11008, 256);     // few rows under a wide head
    calls(20000, 56, 64, 64, 256);                                                           // and many under a narrow one
    calls(20000, 56, 65, 64, 64);
    calls(74897, 56, 64, 64, 64);                                                            // the most rows of the direct route
}
void bounds() {
    check_bounds = true;
    const int heads[][2] = {{256, 256}, {512, 768}, {256, 5120}, {3072, 768}, {768, 2304}, {1024, 11008}, {4096, 11008}, {8192, 28672},
                            {256, 32768}, {256, 33024}, {256, 65536}, {256, 65792}, {512, 131072}, {65792, 256}, {256, 1 << 20}};
    const int rows[][2] = {{1, 1}, {1, 56}, {12, 56}, {37, 56}, {96, 56}, {147, 56}, {768, 56}, {2048, 56}, {4096, 16}, {5, 1000}, {65793, 1}};
    for (const auto& h : heads)
        for (const auto& r : rows)
            for (int panel : {0, 1, 3000})
                bf16_calls(r[0], r[1], h[0], h[1], panel, [&](const Step& c) { expect(run(c), PCM_OK); });
    for (const auto& h : heads)                   // rows beyond the tiles of the widest of those heads
        bf16_calls(1 << 20, 16, h[0], h[1], 0, [&](const Step& c) { expect(run(c), PCM_OK); });
    f32_calls([](const Step& c) { expect(run(c), PCM_OK); });
    if (products < 10000 || sums < 1000) unknown("too few launches were looked at");
}
// The shortest workspace that a call accepts is that of the direct route: whatever the query says, it is enough for every option of the
// shape, and nothing reaches beyond it.
void least() {
    check_bounds = true;
    f32_calls([](const Step& c) {
        check_bounds = false;
        Step plain = c;
        plain.composed = plain.chunk_ratio = false;
        expect(run(plain), PCM_OK);
        size_t enough = query, little = 0;
        while (enough - little > 1) {
            const size_t middle = little + (enough - little) / 2;
            (run(plain, middle) == PCM_OK ? enough : little) = middle;
        }
        check_bounds = true;
        expect(run(c, enough), PCM_OK);
        expect(run(c, enough - 1), PCM_EWORKSPACE);
    });
    const Step large{PCM_F32, 74898, 56, 64, 64, 64, true, true, false, false, false, false, false, 0.f, 0};     // beyond that route
    expect(run(large), PCM_OK);
    expect(run(large, query - 1), PCM_EWORKSPACE);
}
void errors() {
    auto each_launch = [&](const Step& c) {
        fail_at = -1;
        expect(run(c), PCM_OK);
        const int n = launches;
        for (fail_at = 0; fail_at < n; ++fail_at) {
            const int rc = run(c);
            if (rc != PCM_EHIP) call += ", launch " + std::to_string(fail_at) + " of " + std::to_string(n) + " failed";
            expect(rc, PCM_EHIP);
        }
    };
    bf16_calls(37, 56, 512, 768, 0, each_launch);
    bf16_calls(37, 56, 512, 768, 600, each_launch);
    for (int q = 0; q < 16; ++q)
        each_launch(Step{PCM_F32, 46, 56, 64, 96, 32, (q & 1) != 0, (q & 2) != 0, (q & 4) != 0, (q & 8) != 0, false, false, false, 0.f, 0});
}

}  // namespace

int main(int argc, char** argv) {
    if (argc != 2) return 2;
    if (!strcmp(argv[1], "bounds")) bounds();
    else if (!strcmp(argv[1], "errors")) errors();
    else if (!strcmp(argv[1], "least")) least();
    else return 2;
    printf("%d products, %d sums, %d failures\n", products, sums, failures);
    return failures != 0;
}
