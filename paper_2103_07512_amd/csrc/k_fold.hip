// k_fold.hip -- constant folding: every variable-free subtree that a
// variable-dependent node or a root uses is evaluated once on the device and
// enters the programs as a constant: in one launch of one workgroup where the
// nodes are few, else in one launch per subtree height.
#include <hip/hip_runtime.h>
#include <math.h>

#include "ops_device.h"
#include "tgp_internal.h"

namespace tgp {

// Operator op of folded operands, with the interpreter's own FP32 operators
// (ops_device.h, built with the same flags, so a folded value is bitwise the
// value every case computes).
__device__ __forceinline__ float fold_op(int op, float a, float b, float c) {
    float r;
    switch (op) {
    case TGP_ADD: r = f_add(a, b); break;
    case TGP_SUB: r = f_sub(a, b); break;
    case TGP_MULT: r = f_mult(a, b); break;
    case TGP_DIV: r = f_div(a, b); break;
    case TGP_SIN: r = f_sin(a); break;
    case TGP_COS: r = f_cos(a); break;
    case TGP_TAN: r = f_tan(a); break;
    case TGP_EXP: r = f_exp(a); break;
    case TGP_LOG: r = f_log(a); break;
    case TGP_POW: r = f_pow(a, b); break;
    case TGP_MIN: r = f_min(a, b); break;
    case TGP_MAX: r = f_max(a, b); break;
    case TGP_MDIST: r = f_mdist(a, b); break;
    case TGP_NEG: r = f_neg(a); break;
    case TGP_SQRT: r = f_sqrt(a); break;
    case TGP_SIGN: r = f_sign(a); break;
    case TGP_ABS: r = f_abs(a); break;
    case TGP_CLIP: r = f_clip(a, b, c); break;
    case TGP_MOD: r = f_mod(a, b); break;
    case TGP_FRAC: r = f_frac(a); break;
    case TGP_IF: r = f_if(a, b, c); break;
    case TGP_STEP: r = f_step(a); break;
    case TGP_SSTEP: r = f_sstep(a); break;
    case TGP_SSTEPP: r = f_sstepp(a); break;
    case TGP_LEN: r = f_len(a, b); break;
    case TGP_LERP: r = f_lerp(a, b, c); break;
    case TGP_OR: r = f_bitop(a, b, 0); break;
    case TGP_XOR: r = f_bitop(a, b, 1); break;
    case TGP_AND: r = f_bitop(a, b, 2); break;
    case TGP_WARP: r = a; break;  // a constant source reads the same everywhere
    default: r = __builtin_nanf(""); break;
    }
    return r;
}

// A constant node's value: NaNs enter as quiet ones (ops_device.h, min/max).
__device__ __forceinline__ float constant(float v) { return v == v ? v : __builtin_nanf(""); }

// The operator nodes of one height whose subtrees hold no variable, over the
// DAGs of a batch: entry i of list is (DAG, node).  An operator child's value
// comes from the DAG's val, written by the launches of lower heights, a
// constant child's from the node values.
__global__ void k_fold_level(const FoldDesc *jobs, const int2 *list, int32_t n) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int2 e = list[i];
    const FoldDesc J = jobs[e.x];
    const int32_t u = e.y;
    const int32_t *node_kid = J.node_kid;
    const float *node_value = J.node_value;
    float *val = J.val;
    const int32_t *node_op = J.node_op;
    const int op = (int)((uint32_t)node_op[u] & 0xffu);
    const int32_t *k = node_kid + 3 * (int64_t)u;
    auto child = [&](int32_t c) {
        if (c < 0) return 0.0f;
        if (((uint32_t)node_op[c] & 0xffu) != TGP_CONST) return val[c];
        return constant(node_value[c]);
    };
    const float a = child(k[0]);
    const float b = child(k[1]);
    const float c = child(k[2]);
    val[u] = fold_op(op, a, b, c);
}

// All folded nodes of one DAG, ascending in height, by one workgroup.  What
// bounds the launches above for a population of some hundred nodes is their
// number and the copies around them (an upload, one launch for each of four to
// ten heights, a read-back: each some 5 us, their work below 2), so this one
// reads the list from host memory and writes the values there, and between
// heights is a barrier.  A node's operands are read once up front; a folded
// operand is a place in the list (through pos, one entry per DAG node), whose
// value stays in LDS.
__global__ __launch_bounds__(1024) void k_fold_all(const int32_t *node_op, const float *node_value,
                                                   const int32_t *node_kid, int32_t *pos, const int32_t *list,
                                                   int32_t n, const int32_t *first, int32_t heights, float *out) {
    __shared__ uint32_t op[kFoldNodes];       // opcode, bit 8 + j: operand j is a place
    __shared__ uint32_t arg[3][kFoldNodes];   // a place or a value
    __shared__ float val[kFoldNodes];
    __shared__ int32_t start[kFoldHeights + 1];
    const int tid = threadIdx.x;
    for (int h = tid; h <= heights; h += 1024) start[h] = first[h];
    for (int i = tid; i < n; i += 1024) {
        const int32_t u = list[i];
        op[i] = (uint32_t)node_op[u] & 0xffu;
        for (int j = 0; j < 3; ++j) arg[j][i] = (uint32_t)node_kid[3 * (int64_t)u + j];
        pos[u] = i;
    }
    __syncthreads();
    for (int i = tid; i < n; i += 1024)
        for (int j = 0; j < 3; ++j) {
            const int32_t c = (int32_t)arg[j][i];
            uint32_t a = 0;
            if (c >= 0 && ((uint32_t)node_op[c] & 0xffu) == TGP_CONST) a = __float_as_uint(constant(node_value[c]));
            else if (c >= 0) {
                a = (uint32_t)pos[c];
                op[i] |= 256u << j;
            }
            arg[j][i] = a;
        }
    for (int h = 0; h < heights; ++h) {
        __syncthreads();
        for (int i = start[h] + tid; i < start[h + 1]; i += 1024) {
            const uint32_t o = op[i];
            float v[3];
            for (int j = 0; j < 3; ++j) v[j] = o & (256u << j) ? val[arg[j][i]] : __uint_as_float(arg[j][i]);
            const float r = fold_op((int)(o & 0xffu), v[0], v[1], v[2]);
            val[i] = r;
            out[i] = r;
        }
    }
}

hipError_t launch_fold_all(const FoldDesc &d, const int32_t *list, int32_t n, const int32_t *first, int32_t heights,
                           float *out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (n > kFoldNodes || heights > kFoldHeights) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_fold_all, dim3(1), dim3(1024), 0, s, d.node_op, d.node_value, d.node_kid,
                       reinterpret_cast<int32_t *>(d.val), list, n, first, heights, out);
    return hipGetLastError();
}

hipError_t launch_fold_level(const FoldDesc *jobs, const int2 *list, int32_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fold_level, dim3((n + 255) / 256), dim3(256), 0, s, jobs, list, n);
    return hipGetLastError();
}

}  // namespace tgp
