// Value Model formulas (Sec. 5.2): per-task scores of many items are combined into one score
// each by a user formula with conditions.  The formula tree arrives flattened in postfix order
// in the kernel arguments; every workgroup copies it to LDS once (entries of a structure in the
// kernel arguments can only be read with constant indices: a loop over them would make the compiler
// copy the structure to private memory, per lane, and fetch every entry from there).  One thread
// evaluates the formula for four items; the top of its stack stays in registers, the rest lies in
// LDS (one column per thread).  Bound by HBM: 4 * n_tasks bytes read and 4 written per item.
//   code: 0 TASK t  1 CONST c  2 ADD  3 SUB  4 MUL  5 MIN  6 MAX  7 GT (1.0f / 0.0f)  8 SELECT (c != 0 ? x : y); every
//   arithmetic step rounds once.
// What an entry costs is its decoding and its way through the stack, not its arithmetic, so the host folds leaves into
// the operations they feed (vm_fold): "leaf leaf operation" is one step, and so is "operation with a leaf on its right".
// 10 M items x 4 tasks, 24 entries (11 steps): 59 us with a step to every entry, 47 so.
#pragma once

#include "st_device.h"

namespace st {

constexpr int kVmOps = 64;     // entries of a formula, at most
constexpr int kVmDepth = 16;   // stack depth, at most (checked on the host)
constexpr int kVmThreads = 256;

// A step: push the leaf `a` (if any), then run the operation (if any) with the leaf `b` (if any) as its right operand.
// Leaves: 0 none, 1 the constant, 2 + t the score of task t.
struct VmProgram {
    int32_t n_steps;
    int32_t code[kVmOps];  // operation (0: none) | a << 8 | b << 16
    float ca[kVmOps], cb[kVmOps];
};

// A checked formula's steps (n_ops <= kVmOps).
inline void vm_fold(const int32_t* ops, const float* consts, int n_ops, VmProgram* out)
{
    int n = 0;
    auto push_only = [&](int i) { return i >= 0 && (out->code[i] & 255) == 0; };
    for (int i = 0; i < n_ops; ++i) {
        const int op = ops[i] & 255;
        int at = n++;
        out->code[at] = op > 1 ? op : (op == 1 ? 1 : 2 + (ops[i] >> 8)) << 8;
        out->ca[at] = op == 1 ? consts[i] : 0.0f;
        out->cb[at] = 0.0f;
        if (op <= 1 || !push_only(at - 1)) continue;
        // the entry in front is a leaf: the right operand; and if there is one in front of that, it is pushed here
        out->code[at - 1] = op | (out->code[at - 1] >> 8 & 255) << 16;
        out->cb[at - 1] = out->ca[at - 1];
        out->ca[at - 1] = 0.0f;
        n = at--;
        if (!push_only(at - 1)) continue;
        out->code[at - 1] |= out->code[at];
        out->cb[at - 1] = out->cb[at];
        n = at;
    }
    out->n_steps = n;
}

// kVmItems items per thread, in groups of four (one float4 each): the decoding of an entry (its
// read from LDS, the branch on its code) is shared by all of them.
#ifndef ST_VM_ITEMS
#define ST_VM_ITEMS 4
#endif
constexpr int kVmItems = ST_VM_ITEMS;
constexpr int kVmQuads = kVmItems / 4;
static_assert(kVmItems % 4 == 0, "items per thread come in float4 groups");

// LDS of a launch: the stack below the register-held top (depth - 1 elements per thread, at
// least one), then the formula's entries
constexpr int vm_lds_slots(int depth) { return depth > 1 ? depth - 1 : 1; }
constexpr size_t vm_lds_bytes(int depth)
{
    return (size_t)vm_lds_slots(depth) * kVmQuads * kVmThreads * sizeof(float4) + kVmOps * sizeof(int4);
}
static_assert(vm_lds_bytes(kVmDepth) <= 160 * 1024, "the deepest formula fits the LDS of a compute unit");

__global__ __launch_bounds__(kVmThreads) void value_model_kernel(const float* __restrict__ scores, int64_t n,
                                                                 int32_t n_tasks, VmProgram prog,
                                                                 int32_t slots, float* __restrict__ out)
{
    // [slots][kVmQuads][kVmThreads]: sized by the launch from the depth the formula reaches, so that short formulas leave room for many workgroups
    extern __shared__ float4 vm_stack[];
    float4 (*s_stack)[kVmQuads][kVmThreads] = reinterpret_cast<float4 (*)[kVmQuads][kVmThreads]>(vm_stack);
    int4* s_prog = reinterpret_cast<int4*>(vm_stack + (size_t)slots * kVmQuads * kVmThreads);  // {code, bits of the constants}
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i0 = 0; i0 < kVmOps; i0 += 16)
            if (i0 < prog.n_steps)
#pragma unroll
                for (int i = i0; i < i0 + 16; ++i) s_prog[i] = make_int4(prog.code[i], __float_as_int(prog.ca[i]), __float_as_int(prog.cb[i]), 0);
    }
    __syncthreads();
    const int tid = threadIdx.x;
    const int64_t n_sets = (n + kVmItems - 1) / kVmItems;
    const bool aligned_in = (n_tasks & 3) == 0 && (reinterpret_cast<uintptr_t>(scores) & 15) == 0;
    const bool aligned_out = (reinterpret_cast<uintptr_t>(out) & 15) == 0;
    for (int64_t st = (int64_t)blockIdx.x * kVmThreads + tid; st < n_sets; st += (int64_t)gridDim.x * kVmThreads) {
        const int64_t it0 = st * kVmItems;
        // rows of the thread's items (past the end the last item is repeated; those results are not stored)
        const float* row[kVmItems];
#pragma unroll
        for (int u = 0; u < kVmItems; ++u) row[u] = scores + (it0 + u < n ? it0 + u : n - 1) * n_tasks;
        // Rows of up to eight scores are fetched once, with 16-byte loads where they line up: a
        // push per task would otherwise be a load whose 64 lanes touch 64 different lines.
        float tv[kVmItems][8];
        const bool cached = n_tasks <= 8;
        if (cached) {
            if (aligned_in) {
#pragma unroll
                for (int u = 0; u < kVmItems; ++u)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (h * 4 < n_tasks) v = reinterpret_cast<const float4*>(row[u])[h];
                        tv[u][h * 4 + 0] = v.x; tv[u][h * 4 + 1] = v.y; tv[u][h * 4 + 2] = v.z; tv[u][h * 4 + 3] = v.w;
                    }
            } else {
#pragma unroll
                for (int u = 0; u < kVmItems; ++u)
#pragma unroll
                    for (int t = 0; t < 8; ++t) tv[u][t] = t < n_tasks ? row[u][t] : 0.0f;
            }
        }
        // A leaf for items 4g .. 4g+3.  It is the same in every lane, so the switch is a scalar branch;
        // the (empty) assembly statement in every case keeps the compiler from folding the cases into
        // one access indexed by t, which would move the rows from registers to private memory.
        auto leaf4 = [&](int leaf, float c, int g) __attribute__((always_inline)) {
            float4 r;
#define VMK_CASE(k)                                                                               \
    case 2 + k:                                                                                   \
        r = make_float4(tv[4 * g][k], tv[4 * g + 1][k], tv[4 * g + 2][k], tv[4 * g + 3][k]);      \
        asm volatile("; task " #k);                                                               \
        break;
            if (leaf == 1) return make_float4(c, c, c, c);
            if (!cached) {
                const int t = leaf - 2;
                return make_float4(row[4 * g][t], row[4 * g + 1][t], row[4 * g + 2][t], row[4 * g + 3][t]);
            }
            switch (leaf) {
                VMK_CASE(0) VMK_CASE(1) VMK_CASE(2) VMK_CASE(3) VMK_CASE(4) VMK_CASE(5) VMK_CASE(6)
            default:
                r = make_float4(tv[4 * g][7], tv[4 * g + 1][7], tv[4 * g + 2][7], tv[4 * g + 3][7]);
                break;
            }
#undef VMK_CASE
            return r;
        };
        // Element e of the stack lies in s_stack[e] while it is not the top; the top is `tos`.
        int top = 0;  // elements on the stack (the same in every lane, like everything decoded below)
        float4 tos[kVmQuads];
#pragma unroll
        for (int g = 0; g < kVmQuads; ++g) tos[g] = make_float4(0.f, 0.f, 0.f, 0.f);
        int4 e = s_prog[0];
        for (int i = 0; i < prog.n_steps; ++i) {
            const int step = __builtin_amdgcn_readfirstlane(e.x);
            const float ca = __int_as_float(__builtin_amdgcn_readfirstlane(e.y)), cb = __int_as_float(__builtin_amdgcn_readfirstlane(e.z));
            const int code = step & 255, la = step >> 8 & 255, lb = step >> 16;
            e = s_prog[i + 1 < kVmOps ? i + 1 : i];  // the next step, while this one runs
            if (la) {
                if (top > 0) {
#pragma unroll
                    for (int g = 0; g < kVmQuads; ++g) s_stack[top - 1][g][tid] = tos[g];
                }
                ++top;
#pragma unroll
                for (int g = 0; g < kVmQuads; ++g) tos[g] = leaf4(la, ca, g);
            }
            if (code == 0) continue;
            // operands: x under y; y is the leaf or the top, x the top or the element below
            float4 a[kVmQuads], y[kVmQuads];
            if (lb) {
#pragma unroll
                for (int g = 0; g < kVmQuads; ++g) {
                    a[g] = tos[g];
                    y[g] = leaf4(lb, cb, g);
                }
            } else {
                --top;
#pragma unroll
                for (int g = 0; g < kVmQuads; ++g) {
                    a[g] = s_stack[top - 1][g][tid];
                    y[g] = tos[g];
                }
            }
            if (code == 8) {
                --top;
#pragma unroll
                for (int g = 0; g < kVmQuads; ++g) {
                    const float4 c = s_stack[top - 1][g][tid];
                    tos[g] = make_float4(c.x != 0.0f ? a[g].x : y[g].x, c.y != 0.0f ? a[g].y : y[g].y, c.z != 0.0f ? a[g].z : y[g].z,
                                         c.w != 0.0f ? a[g].w : y[g].w);
                }
            } else {
#define VMK_EACH(EXPR)                                                                              \
    _Pragma("unroll") for (int g = 0; g < kVmQuads; ++g)                                              \
    {                                                                                                 \
        const float4 x = a[g], z = y[g];                                                              \
        tos[g] = make_float4(EXPR(x.x, z.x), EXPR(x.y, z.y), EXPR(x.z, z.z), EXPR(x.w, z.w));         \
    }
#define VMK_MIN(p, q) ((p) < (q) ? (p) : (q))
#define VMK_MAX(p, q) ((p) > (q) ? (p) : (q))
#define VMK_GT(p, q) ((p) > (q) ? 1.0f : 0.0f)
                switch (code) {
                case 2: VMK_EACH(__fadd_rn) break;
                case 3: VMK_EACH(__fsub_rn) break;
                case 4: VMK_EACH(__fmul_rn) break;
                case 5: VMK_EACH(VMK_MIN) break;
                case 6: VMK_EACH(VMK_MAX) break;
                default: VMK_EACH(VMK_GT) break;
                }
#undef VMK_EACH
#undef VMK_MIN
#undef VMK_MAX
#undef VMK_GT
            }
        }
#pragma unroll
        for (int g = 0; g < kVmQuads; ++g) {
            const float4 r = tos[g];
            const int64_t i0 = it0 + 4 * g;
            if (i0 + 3 < n && aligned_out) {
                *reinterpret_cast<float4*>(out + i0) = r;
            } else {
                if (i0 < n) out[i0] = r.x;
                if (i0 + 1 < n) out[i0 + 1] = r.y;
                if (i0 + 2 < n) out[i0 + 2] = r.z;
                if (i0 + 3 < n) out[i0 + 3] = r.w;
            }
        }
    }
}

}  // namespace st
