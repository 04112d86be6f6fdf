// A device made of host memory, for CPU checks of the library's host side (which
// launch shape a call takes, which tables and vectors it holds, what it does when
// memory is short): the HIP calls that the host code makes, over calloc and a
// byte count that a check may limit, and every kernel launcher as an empty
// function.  Launchers whose arguments a check looks at call a hook.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>

#include "../paper_2209_00806_amd/csrc/tbpm_engine.h"

namespace fake {
size_t total = (size_t)1 << 40, used = 0;
size_t hidden = 0;  // bytes that hipMemGetInfo holds back (taken by others)
std::map<void *, size_t> blocks;
int uploads = 0;              // synchronous copies to the device
std::function<void(const tbpm::InitParams &)> on_init;
std::function<void(int64_t n_el, int64_t n_used)> on_qe_accum;
std::function<void(int log2s, int log2sb)> on_qe_finalize;
std::function<void(const tbpm::ChainParams &, bool fp32)> on_chain, on_wide;
std::function<void(bool fp32, int n_tiles)> on_values;
std::function<void(int width, int max_eval, int max_stage, const tbpm::ChainParams &)> on_hay;
std::function<void(bool fp32)> on_pass;
// rows that a launch reads or writes of a buffer lie inside one block of memory
inline bool holds(const void *p, size_t bytes) {
    auto it = blocks.upper_bound((void *)p);
    if (it == blocks.begin()) return false;
    --it;
    return (char *)p + bytes <= (char *)it->first + it->second;
}
}  // namespace fake

extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
    if (fake::used + n > fake::total) {
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    *p = std::calloc(1, n ? n : 1);
    if (!*p) return hipErrorOutOfMemory;
    fake::blocks[*p] = n;
    fake::used += n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    auto it = fake::blocks.find(p);
    if (it == fake::blocks.end()) return p ? hipErrorInvalidValue : hipSuccess;
    fake::used -= it->second;
    fake::blocks.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    *p = std::calloc(1, n ? n : 1);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *f, size_t *t) {
    const size_t taken = fake::used + fake::hidden;
    *f = taken < fake::total ? fake::total - taken : 0;
    *t = fake::total;
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind kind) {
    fake::uploads += kind == hipMemcpyHostToDevice;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) {
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    *g = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *g, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    *g = reinterpret_cast<hipGraphExec_t>(1);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
    *a = hipPointerAttribute_t{};
    a->type = fake::holds(p, 1) ? hipMemoryTypeDevice : hipMemoryTypeHost;
    return hipSuccess;
}
}  // extern "C"

namespace tbpm {
#define OK_ \
    { return hipSuccess; }
hipError_t launch_pass(int, bool fp32, bool, bool, int, int, const PassParams &, hipStream_t) {
    if (fake::on_pass) fake::on_pass(fp32);
    return hipSuccess;
}
hipError_t launch_pass_staged(int, bool fp32, bool, bool, int, bool, const PassParams &, hipStream_t) {
    if (fake::on_pass) fake::on_pass(fp32);
    return hipSuccess;
}
hipError_t launch_init(bool, const InitParams &p, hipStream_t) {
    if (fake::on_init) fake::on_init(p);
    return hipSuccess;
}
// norms of one, which the check after a run expects
hipError_t launch_reduce(int n_inst, int, const ReduceParams &p, hipStream_t) {
    if (p.norm2_all)
        for (int64_t i = 0; i < (int64_t)n_inst * p.n_steps * p.s_user; ++i) p.norm2_all[i] = 1.0;
    return hipSuccess;
}
hipError_t launch_dos(const double *, int32_t, int32_t, double, int, double *, double *, hipStream_t) OK_
hipError_t launch_dos_backward(const double *, int32_t, int32_t, double, int, double *, hipStream_t) OK_
hipError_t launch_convert_values(const DevMatrix &, const double *, const double *, int64_t, hipStream_t) OK_
hipError_t launch_copy(const void *, void *, size_t, hipStream_t) OK_
hipError_t launch_adjoint_pair(int, bool, int, const AdjPairParams &, hipStream_t) OK_
hipError_t launch_adjoint_pass(int, bool, const AdjParams &, hipStream_t) OK_
hipError_t launch_pair(int, bool fp32, bool, bool, int, const FusedParams &, hipStream_t) {
    if (fake::on_pass) fake::on_pass(fp32);
    return hipSuccess;
}
hipError_t launch_chain(bool fp32, bool, int, int, int, int, const ChainParams &p, hipStream_t) {
    if (fake::on_chain) fake::on_chain(p, fp32);
    return p.depth >= 1 && p.depth <= p.table_depth ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_chain_cheb(int, bool, int, int, int, int, const ChainParams &p, const ChainCheb &, hipStream_t) {
    if (fake::on_chain) fake::on_chain(p, false);
    return p.depth >= 1 && p.depth <= p.table_depth ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_pass_wide(bool fp32, int, int, int, const ChainParams &p, hipStream_t) {
    if (fake::on_wide) fake::on_wide(p, fp32);
    return hipSuccess;
}
hipError_t launch_chain_values(bool fp32, bool, const ChainTileTab &, int32_t n_tiles, const DevMatrix &, void *,
                               void *, hipStream_t) {
    if (fake::on_values) fake::on_values(fp32, n_tiles);
    return hipSuccess;
}
hipError_t launch_chain_reduce(int, int, int64_t, const ReduceParams &, int32_t *, bool, hipStream_t) OK_
hipError_t launch_qe_accum(bool, const void *, double *, int64_t n_el, int64_t n_used, const double *, int32_t,
                           const int32_t *, int32_t, int32_t, int64_t, hipStream_t) {
    if (fake::on_qe_accum) fake::on_qe_accum(n_el, n_used);
    return hipSuccess;
}
int32_t qe_partial_blocks(int64_t) { return 4; }
hipError_t launch_qe_finalize(const double *, int64_t, int32_t log2s, int32_t log2sb, int32_t, int32_t,
                              const int32_t *, double *, double *, double *, hipStream_t) {
    if (fake::on_qe_finalize) fake::on_qe_finalize(log2s, log2sb);
    return hipSuccess;
}
hipError_t launch_gather_values(const int64_t *, int64_t, const double *, double *, hipStream_t) OK_
hipError_t launch_join(const double *, const double *, int64_t, int32_t, int32_t, int32_t, int32_t, double *,
                       hipStream_t) OK_
hipError_t launch_pack(const double *, const double *, int64_t, int32_t, int32_t, const int32_t *, double *,
                       hipStream_t) OK_
hipError_t launch_jcorr(bool, const TileDesc *, int32_t, int32_t, int32_t, int32_t, int64_t, const void *,
                        const uint32_t *, const int32_t *, const double *, double *, int32_t, int64_t, int64_t,
                        hipStream_t) OK_
// 1500 coefficients, from 16384 samples on
hipError_t launch_fermi_cheb(double, double, double, int32_t n, double, double *, double *, int32_t *last, hipStream_t) {
    *last = n >= 16384 ? 1499 : n / 2 - 1;
    return hipSuccess;
}
hipError_t launch_ac_cond(const double *, int32_t, int32_t, double, double, double, int, double *, double *,
                          hipStream_t) OK_
hipError_t launch_ac_kk(const double *, int32_t, double *, hipStream_t) OK_
hipError_t launch_hay_spmv(bool, const TileDesc *, int32_t, int32_t, int32_t, const int32_t *, const void *,
                           const uint32_t *, int32_t, const double *, const double *, const double *, double *,
                           const double *, int32_t *, double *, hipStream_t) OK_
hipError_t launch_hay_axpy(const TileDesc *, int32_t, int32_t, int32_t, int32_t, const double *, const double *,
                           double *, const double *, double *, hipStream_t) OK_
int32_t hay_fold_count(int32_t) { return 0; }
hipError_t launch_hay_reduce(const double *, int32_t, int32_t, int32_t, int32_t, double, double *, int32_t *, int32_t,
                             double *, double *, double *, hipStream_t) OK_
hipError_t launch_hay_step(bool, int width, int max_eval, int max_stage, ChainParams p, const double *, hipStream_t) {
    if (fake::on_hay) fake::on_hay(width, max_eval, max_stage, p);
    if (fake::on_chain) fake::on_chain(p, false);
    return hipSuccess;
}
hipError_t launch_hay_reduce3(const double *, int32_t, int32_t, bool, double, double *, int32_t *, int32_t, double *,
                              double *, hipStream_t) OK_
hipError_t launch_hay_ldos(const double *, const double *, int32_t, int32_t, const double *, int64_t, double, double *,
                           hipStream_t) OK_
int32_t kpm_max_moments_lds() { return 2048; }
KpmProductShape kpm_product_shape(int32_t) { return {4, 4, 2, 0}; }
hipError_t launch_kpm_product(int32_t, const double *, const double *, int64_t, int64_t, int32_t, int32_t, int64_t,
                              int32_t, double *, hipStream_t) OK_
hipError_t launch_kpm_sum_parts(const double *, int64_t, int32_t, int64_t, double, double *, hipStream_t) OK_
hipError_t launch_kubo_bastin(const double *, int32_t, double, double, double, int32_t, const double *, int32_t, double,
                              double, double *, double *, double *, hipStream_t) OK_
hipError_t launch_expand_states(const double *, const int32_t *, int32_t, double *, int32_t, int64_t, hipStream_t) OK_
hipError_t launch_lam_init(double *, const double *, const double *, int32_t, int32_t, int64_t, hipStream_t) OK_
hipError_t launch_fill_zero(double *, int64_t, hipStream_t) OK_
hipError_t launch_grad_scatter(const void *, const double *, const int64_t *, int64_t, bool, double, double *, double *,
                               const int32_t *, int64_t, const int32_t *, int32_t, hipStream_t) OK_
tbpm_status propagate_noalloc(tbpm_hamiltonian *, const double *, int32_t, int32_t, double, double, double, bool,
                              double *, double *, hipStream_t) {
    return TBPM_OK;
}
size_t noalloc_scratch_bytes() { return 0; }
#undef OK_
}  // namespace tbpm
