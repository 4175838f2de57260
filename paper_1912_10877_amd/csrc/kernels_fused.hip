// Fused tile-pass kernels: forward sweep and reversible adjoint sweep.
//
// One workgroup owns one tile: 2^t elements = Bc = 2^c consecutive batch slots (lowest tile
// bits) x the 2^(t-c) amplitudes spanned by the pass's tile qubits, with every other qubit
// fixed by the tile id. The tile is staged in LDS (XOR-swizzled), then processed in register
// groups: each of the 2^(t-RB) threads holds the 2^RB elements that differ only in the
// group's RB register bits, so a one-qubit gate on a register bit is pure ALU work on pairs of
// registers. Gates of 2 or 3 qubits are applied directly in LDS. The backward kernel holds psi
// (complex128: the FP64 uncompute) and lambda (widened to FP64 in registers) and, per gate,
// first adds 2 Re <lambda|M|psi> over the tile (eq. outer-product reduced to the parameter),
// then applies U^dagger to both (eq. apply-back). Per-thread gradient partials go to LDS and
// are reduced once per register group, in a fixed order.
//
// The op records are read where they lie, through the scalar cache; the record of the next op is
// fetched while the current op computes.
#include <algorithm>
#include <cmath>
#include <map>
#include <tuple>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "fused.h"

namespace yao {

namespace {
struct ZBatch {
    const ZSlot* zs = nullptr;
    int nz = 0;
};
ZBatch g_zbatch;
}  // namespace

void set_zbatch(const ZSlot* zs, int nz)
{
    g_zbatch.zs = nz > 0 ? zs : nullptr;
    g_zbatch.nz = nz > 0 ? nz : 0;
}

int zbatch_count()
{
    return g_zbatch.zs ? g_zbatch.nz : 1;
}

const ZSlot* zbatch_slots()
{
    return g_zbatch.zs;
}

namespace {

struct PassArgs {
    void* psi;
    void* lam;
    const POp* ops;         // the pass's records: ops[0 .. nops)
    const PGroupDesc* groups;  // the pass's groups: groups[0 .. ngroups), op0 relative to ops
    const double* mats;
    double* gpartial;       // [slot][B][pstride]
    int n, B, c, t;
    int ngroups, nops;
    int ntq, nnt;
    int ntiles;
    int pstride;
    int tile_qubits[kMaxTileBits];
    int nontile_qubits[40];
    uint64_t rofs[1 << kMaxRegBits];  // element offset (x B) of load register r from the thread's first
    const uint4* dmats;     // the pass's dense block matrices (forward), staged in LDS
    int ndm;                // their size in 16-byte words
    // Store permutation: stored tile element e = th + r * nthr comes from LDS tile element
    // store_thread_bits(th) | sreg[r] (thread bit i of e moves to tile bit ssrc[i]).
    int ssrc[kMaxTileBits];
    uint32_t sreg[1 << kMaxRegBits];
    int mslots;             // reverse passes: gradient-carrying ops per register group (at most)
    // Launches over several circuits of one structure (grid z): circuit z's state, adjoint
    // state, records (ops: program base, plus op_first) and partial sums; null: one circuit.
    const ZSlot* zs;
    int op_first;
};

// The per-circuit pointers of a launch (the circuit's own, or its z slot's).
template <typename A> __device__ __forceinline__ void* z_psi(const A& a)
{
    return a.zs ? a.zs[blockIdx.z].psi : a.psi;
}
template <typename A> __device__ __forceinline__ void* z_lam(const A& a)
{
    return a.zs ? a.zs[blockIdx.z].lam : a.lam;
}
template <typename A> __device__ __forceinline__ const POp* z_ops(const A& a)
{
    return a.zs ? a.zs[blockIdx.z].ops + a.op_first : a.ops;
}
template <typename A> __device__ __forceinline__ double* z_partial(const A& a, double* p)
{
    return a.zs ? a.zs[blockIdx.z].partial : p;
}

__device__ __forceinline__ uint32_t swz(uint32_t e)
{
    return e ^ (((e >> 4) ^ (e >> 8)) & 15u);
}

template <typename V, typename RR> __device__ __forceinline__ V mkv(RR a, RR b)
{
    V v;
    v.x = a;
    v.y = b;
    return v;
}

__device__ __forceinline__ int sc(int v)
{
    return __builtin_amdgcn_readfirstlane(v);
}
__device__ __forceinline__ uint64_t sc64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Control fields of an op record, made wave-uniform (scalar registers).
struct OpCtl {
    int type, gen, rpos, slot, mat, var;
    uint32_t cmask, cval;
    uint64_t omask, oval;
};
// Control fields and the one-qubit matrix of an op, wave-uniform. The matrix is read in the
// precision MR: the host stores float entries (u viewed as float[8]) in programs for complex64
// forward sweeps, double entries otherwise.
template <typename MR> struct OpS {
    OpCtl c;
    MR m[8];  // re[4], im[4]
};
// Op records and group descriptors are read in place through the scalar cache: a pointer in
// the constant address space tells the compiler that the kernel never writes them, so
// wave-uniform reads become scalar loads straight into SGPRs (the records are written by the
// host or by the bind kernel before the pass is launched).
#define YAO_CONST __attribute__((address_space(4)))
template <typename T> __device__ __forceinline__ const YAO_CONST T* cptr(const T* p)
{
    return (const YAO_CONST T*)p;
}
__device__ __forceinline__ OpCtl op_ctl_c(const YAO_CONST POp* r)
{
    OpCtl o;
    o.type = r->type;
    o.gen = r->gen;
    o.rpos = r->rpos;
    o.slot = r->slot;
    o.mat = r->mat;
    o.var = r->var;
    o.cmask = r->cmask;
    o.cval = r->cval;
    o.omask = r->omask;
    o.oval = r->oval;
    return o;
}
template <typename MR> __device__ __forceinline__ OpS<MR> load_op_c(const YAO_CONST POp* r)
{
    OpS<MR> o;
    o.c = op_ctl_c(r);
    if constexpr (sizeof(MR) == 4) {
        const YAO_CONST float* f = (const YAO_CONST float*)r->u;
#pragma unroll
        for (int q = 0; q < 8; ++q) o.m[q] = f[q];
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) o.m[q] = r->u[q];
    }
    return o;
}

__device__ __forceinline__ void fold_outer_controls(OpCtl& c, uint64_t base)
{
    if ((base & c.omask) != c.oval) {
        c.cmask = 0x80000000u;
        c.cval = 0x80000000u;
    }
}

// ------------------------------------------------------------------------------ in-place updates
// The common one-qubit updates are written as inline assembly whose results are tied to the
// registers of their inputs. A register group's amplitudes stay in fixed registers from op to
// op; computed as plain expressions, each op variant would leave its results in fresh
// registers and every op would end with a copy of all of them. Scalar operands are the op's
// matrix entries (SGPRs); each VALU instruction reads at most one of them.
#define YAO_IP_FNS(T, V, SFX, MOV)                                                                       \
    /* (a, b) <- (c a + i s b, i s a + c b) */                                                          \
    __device__ __forceinline__ void rx_ip(V& a, V& b, T cc, T ss)                                      \
    {                                                                                                   \
        T t0, t1;                                                                                       \
        asm("v_mul_" SFX " %[t0], %[s], %[by]\n\t"                                                    \
            "v_mul_" SFX " %[t1], %[s], %[ax]\n\t"                                                    \
            "v_fma_" SFX " %[ax], %[c], %[ax], -%[t0]\n\t"                                            \
            "v_fma_" SFX " %[by], %[c], %[by], %[t1]\n\t"                                             \
            "v_mul_" SFX " %[t0], %[s], %[bx]\n\t"                                                    \
            "v_mul_" SFX " %[t1], %[s], %[ay]\n\t"                                                    \
            "v_fma_" SFX " %[ay], %[c], %[ay], %[t0]\n\t"                                             \
            "v_fma_" SFX " %[bx], %[c], %[bx], -%[t1]"                                                  \
            : [ax] "+v"(a.x), [ay] "+v"(a.y), [bx] "+v"(b.x), [by] "+v"(b.y), [t0] "=&v"(t0),            \
              [t1] "=&v"(t1)                                                                            \
            : [c] "s"(cc), [s] "s"(ss));                                                                \
    }                                                                                                   \
    /* a <- (r + i m) a */                                                                              \
    __device__ __forceinline__ void diag_ip(V& a, T r, T m)                                            \
    {                                                                                                   \
        T t0, t1;                                                                                       \
        asm("v_mul_" SFX " %[t0], %[m], %[ay]\n\t"                                                    \
            "v_mul_" SFX " %[t1], %[m], %[ax]\n\t"                                                    \
            "v_fma_" SFX " %[ax], %[r], %[ax], -%[t0]\n\t"                                            \
            "v_fma_" SFX " %[ay], %[r], %[ay], %[t1]"                                                   \
            : [ax] "+v"(a.x), [ay] "+v"(a.y), [t0] "=&v"(t0), [t1] "=&v"(t1)                             \
            : [r] "s"(r), [m] "s"(m));                                                                  \
    }                                                                                                   \
    /* (a, b) <- U (a, b) for U = mr + i mi, row-major; four interleaved FMA chains, the last */  \
    /* of which ends in b.y itself */                                                                 \
    __device__ __forceinline__ void dense_ip(V& a, V& b, const T* mr, const T* mi)                     \
    {                                                                                                   \
        T t0, t1, t2, t3;                                                                               \
        asm("v_mul_" SFX " %[t0], %[r0], %[ax]\n\t"                                                   \
            "v_mul_" SFX " %[t1], %[r0], %[ay]\n\t"                                                   \
            "v_mul_" SFX " %[t2], %[r2], %[ax]\n\t"                                                   \
            "v_mul_" SFX " %[t3], %[r2], %[ay]\n\t"                                                   \
            "v_fma_" SFX " %[t0], -%[i0], %[ay], %[t0]\n\t"                                           \
            "v_fma_" SFX " %[t1], %[i0], %[ax], %[t1]\n\t"                                            \
            "v_fma_" SFX " %[t2], -%[i2], %[ay], %[t2]\n\t"                                           \
            "v_fma_" SFX " %[t3], %[i2], %[ax], %[t3]\n\t"                                            \
            "v_fma_" SFX " %[t0], %[r1], %[bx], %[t0]\n\t"                                            \
            "v_fma_" SFX " %[t1], %[i1], %[bx], %[t1]\n\t"                                            \
            "v_fma_" SFX " %[t2], %[r3], %[bx], %[t2]\n\t"                                            \
            "v_fma_" SFX " %[t3], %[i3], %[bx], %[t3]\n\t"                                            \
            "v_fma_" SFX " %[t0], -%[i1], %[by], %[t0]\n\t"                                           \
            "v_fma_" SFX " %[t1], %[r1], %[by], %[t1]\n\t"                                            \
            "v_fma_" SFX " %[t2], -%[i3], %[by], %[t2]\n\t"                                           \
            "v_fma_" SFX " %[by], %[r3], %[by], %[t3]\n\t"                                            \
            MOV " %[ax], %[t0]\n\t"                                                                   \
            MOV " %[ay], %[t1]\n\t"                                                                   \
            MOV " %[bx], %[t2]"                                                                         \
            : [ax] "+v"(a.x), [ay] "+v"(a.y), [bx] "+v"(b.x), [by] "+v"(b.y), [t0] "=&v"(t0),            \
              [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3)                                            \
            : [r0] "s"(mr[0]), [r1] "s"(mr[1]), [r2] "s"(mr[2]), [r3] "s"(mr[3]), [i0] "s"(mi[0]),       \
              [i1] "s"(mi[1]), [i2] "s"(mi[2]), [i3] "s"(mi[3]));                                        \
    }
#define YAO_IP_CTL_FNS(T, V, SFX, MOV)                                                                   \
    /* (a, b) <- U (a, b) in the lanes of the mask m (a ballot), unchanged elsewhere */                \
    __device__ __forceinline__ void dense_ctl_ip(V& a, V& b, const T* mr, const T* mi, uint64_t m)     \
    {                                                                                                   \
        T t0, t1, t2, t3;                                                                               \
        uint64_t sv;                                                                                    \
        asm volatile("v_mul_" SFX " %[t0], %[r0], %[ax]\n\t"                                          \
                     "v_mul_" SFX " %[t1], %[r0], %[ay]\n\t"                                          \
                     "v_mul_" SFX " %[t2], %[r2], %[ax]\n\t"                                          \
                     "v_mul_" SFX " %[t3], %[r2], %[ay]\n\t"                                          \
                     "v_fma_" SFX " %[t0], -%[i0], %[ay], %[t0]\n\t"                                  \
                     "v_fma_" SFX " %[t1], %[i0], %[ax], %[t1]\n\t"                                   \
                     "v_fma_" SFX " %[t2], -%[i2], %[ay], %[t2]\n\t"                                  \
                     "v_fma_" SFX " %[t3], %[i2], %[ax], %[t3]\n\t"                                   \
                     "v_fma_" SFX " %[t0], %[r1], %[bx], %[t0]\n\t"                                   \
                     "v_fma_" SFX " %[t1], %[i1], %[bx], %[t1]\n\t"                                   \
                     "v_fma_" SFX " %[t2], %[r3], %[bx], %[t2]\n\t"                                   \
                     "v_fma_" SFX " %[t3], %[i3], %[bx], %[t3]\n\t"                                   \
                     "v_fma_" SFX " %[t0], -%[i1], %[by], %[t0]\n\t"                                  \
                     "v_fma_" SFX " %[t1], %[r1], %[by], %[t1]\n\t"                                   \
                     "v_fma_" SFX " %[t2], -%[i3], %[by], %[t2]\n\t"                                  \
                     "v_fma_" SFX " %[t3], %[r3], %[by], %[t3]\n\t"                                   \
                     "s_mov_b64 %[sv], exec\n\t"                                                      \
                     "s_mov_b64 exec, %[m]\n\t"                                                       \
                     MOV " %[ax], %[t0]\n\t"                                                          \
                     MOV " %[ay], %[t1]\n\t"                                                          \
                     MOV " %[bx], %[t2]\n\t"                                                          \
                     MOV " %[by], %[t3]\n\t"                                                          \
                     "s_mov_b64 exec, %[sv]"                                                            \
                     : [ax] "+v"(a.x), [ay] "+v"(a.y), [bx] "+v"(b.x), [by] "+v"(b.y), [t0] "=&v"(t0),   \
                       [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), [sv] "=&s"(sv)                   \
                     : [r0] "s"(mr[0]), [r1] "s"(mr[1]), [r2] "s"(mr[2]), [r3] "s"(mr[3]),              \
                       [i0] "s"(mi[0]), [i1] "s"(mi[1]), [i2] "s"(mi[2]), [i3] "s"(mi[3]), [m] "s"(m));  \
    }
YAO_IP_CTL_FNS(float, float2, "f32", "v_mov_b32")
YAO_IP_CTL_FNS(double, double2, "f64", "v_mov_b64")
#undef YAO_IP_CTL_FNS
YAO_IP_FNS(float, float2, "f32", "v_mov_b32")
YAO_IP_FNS(double, double2, "f64", "v_mov_b64")
#undef YAO_IP_FNS

// Swap a and b in the lanes of the mask m (a ballot, so a subset of the active lanes): exec is
// narrowed to m for the moves and restored.
__device__ __forceinline__ void cswap_ip(float2& a, float2& b, uint64_t m)
{
    uint64_t sv;
    asm volatile("s_mov_b64 %[sv], exec\n\t"
                 "s_mov_b64 exec, %[m]\n\t"
                 "v_swap_b32 %[ax], %[bx]\n\t"
                 "v_swap_b32 %[ay], %[by]\n\t"
                 "s_mov_b64 exec, %[sv]"
                 : [ax] "+v"(a.x), [ay] "+v"(a.y), [bx] "+v"(b.x), [by] "+v"(b.y), [sv] "=&s"(sv)
                 : [m] "s"(m));
}
__device__ __forceinline__ void cswap_ip(double2& a, double2& b, uint64_t m)
{
    uint64_t sv;
    double t;
    asm volatile("s_mov_b64 %[sv], exec\n\t"
                 "s_mov_b64 exec, %[m]\n\t"
                 "v_mov_b64 %[t], %[ax]\n\t"
                 "v_mov_b64 %[ax], %[bx]\n\t"
                 "v_mov_b64 %[bx], %[t]\n\t"
                 "v_mov_b64 %[t], %[ay]\n\t"
                 "v_mov_b64 %[ay], %[by]\n\t"
                 "v_mov_b64 %[by], %[t]\n\t"
                 "s_mov_b64 exec, %[sv]"
                 : [ax] "+v"(a.x), [ay] "+v"(a.y), [bx] "+v"(b.x), [by] "+v"(b.y), [t] "=&v"(t), [sv] "=&s"(sv)
                 : [m] "s"(m));
}
__device__ __forceinline__ void cswap_ip(double2& a, double2& b, double2& c, double2& d, uint64_t m)
{
    uint64_t sv;
    double t;
    asm volatile("s_mov_b64 %[sv], exec\n\t"
                 "s_mov_b64 exec, %[m]\n\t"
                 "v_mov_b64 %[t], %[ax]\n\t"
                 "v_mov_b64 %[ax], %[bx]\n\t"
                 "v_mov_b64 %[bx], %[t]\n\t"
                 "v_mov_b64 %[t], %[ay]\n\t"
                 "v_mov_b64 %[ay], %[by]\n\t"
                 "v_mov_b64 %[by], %[t]\n\t"
                 "v_mov_b64 %[t], %[cx]\n\t"
                 "v_mov_b64 %[cx], %[dx]\n\t"
                 "v_mov_b64 %[dx], %[t]\n\t"
                 "v_mov_b64 %[t], %[cy]\n\t"
                 "v_mov_b64 %[cy], %[dy]\n\t"
                 "v_mov_b64 %[dy], %[t]\n\t"
                 "s_mov_b64 exec, %[sv]"
                 : [ax] "+v"(a.x), [ay] "+v"(a.y), [bx] "+v"(b.x), [by] "+v"(b.y), [cx] "+v"(c.x),
                   [cy] "+v"(c.y), [dx] "+v"(d.x), [dy] "+v"(d.y), [t] "=&v"(t), [sv] "=&s"(sv)
                 : [m] "s"(m));
}

// diag(1, d) on a register bit: the reverse passes' Z-generator diagonal ops, whose first entry
// is carried as a phase of the whole tile.
constexpr int kDiagHigh = 100;

// An uncontrolled one-qubit op of structure TYPE (OT_RX, OT_DIAG, kDiagHigh or OT_DENSE) on
// register bit J.
template <int J, int TYPE, typename RR, typename V, int N>
__device__ __forceinline__ void pairs_ip(V (&x)[N], const RR* mr, const RR* mi)
{
#pragma unroll
    for (int a = 0; a < N; ++a) {
        if (a & (1 << J)) continue;
        V& p = x[a];
        V& q = x[a + (1 << J)];
        if constexpr (TYPE == OT_RX) {
            rx_ip(p, q, mr[0], mi[1]);
        } else if constexpr (TYPE == OT_DIAG) {
            diag_ip(p, mr[0], mi[0]);
            diag_ip(q, mr[3], mi[3]);
        } else if constexpr (TYPE == kDiagHigh) {
            diag_ip(q, mr[3], mi[3]);
        } else {
            dense_ip(p, q, mr, mi);
        }
    }
}

// Any one-qubit op on register bit J (as a dense 2 x 2 matrix) where the pair's tile index
// matches the tile-bit controls (every pair when cmask is 0); the backward form updates psi
// and lambda with the same matrix.
template <int J, typename RR, typename V, int N>
__device__ __forceinline__ void pairs_dense_ctl_ip(V (&x)[N], const RR* mr, const RR* mi, uint32_t ethr,
                                                   const uint32_t (&er)[N], uint32_t cmask, uint32_t cval)
{
#pragma unroll
    for (int a = 0; a < N; ++a) {
        if (a & (1 << J)) continue;
        const uint64_t m = __builtin_amdgcn_ballot_w64(((ethr | er[a]) & cmask) == cval);
        dense_ctl_ip(x[a], x[a + (1 << J)], mr, mi, m);
    }
}
template <int J, int N>
__device__ __forceinline__ void pairs_dense_ctl_ip(double2 (&x)[N], double2 (&y)[N], const double* mr,
                                                   const double* mi, uint32_t ethr, const uint32_t (&er)[N],
                                                   uint32_t cmask, uint32_t cval)
{
#pragma unroll
    for (int a = 0; a < N; ++a) {
        if (a & (1 << J)) continue;
        const uint64_t m = __builtin_amdgcn_ballot_w64(((ethr | er[a]) & cmask) == cval);
        dense_ctl_ip(x[a], x[a + (1 << J)], mr, mi, m);
        dense_ctl_ip(y[a], y[a + (1 << J)], mr, mi, m);
    }
}

// A SWAP of the pair on register bit J where the pair's tile index matches the tile-bit controls.
template <int J, typename V, int N>
__device__ __forceinline__ void pairs_cswap_ip(V (&x)[N], uint32_t ethr, const uint32_t (&er)[N], uint32_t cmask,
                                               uint32_t cval)
{
    if ((cmask & ~er[N - 1]) == 0) {
        // Controls on register bits only (er[N - 1] holds them all): a pair is swapped in
        // every lane or in none, so the pairs that fail them cost nothing.
#pragma unroll
        for (int a = 0; a < N; ++a) {
            if (a & (1 << J)) continue;
            if ((er[a] & cmask) == cval) cswap_ip(x[a], x[a + (1 << J)], __builtin_amdgcn_read_exec());
        }
        return;
    }
#pragma unroll
    for (int a = 0; a < N; ++a) {
        if (a & (1 << J)) continue;
        const uint64_t m = __builtin_amdgcn_ballot_w64(((ethr | er[a]) & cmask) == cval);
        cswap_ip(x[a], x[a + (1 << J)], m);
    }
}
template <int J, int N>
__device__ __forceinline__ void pairs_cswap_ip(double2 (&x)[N], double2 (&y)[N], uint32_t ethr,
                                               const uint32_t (&er)[N], uint32_t cmask, uint32_t cval)
{
    if ((cmask & ~er[N - 1]) == 0) {
        // Controls on register bits only, as above.
#pragma unroll
        for (int a = 0; a < N; ++a) {
            if (a & (1 << J)) continue;
            if ((er[a] & cmask) == cval)
                cswap_ip(x[a], x[a + (1 << J)], y[a], y[a + (1 << J)], __builtin_amdgcn_read_exec());
        }
        return;
    }
#pragma unroll
    for (int a = 0; a < N; ++a) {
        if (a & (1 << J)) continue;
        const uint64_t m = __builtin_amdgcn_ballot_w64(((ethr | er[a]) & cmask) == cval);
        cswap_ip(x[a], x[a + (1 << J)], y[a], y[a + (1 << J)], m);
    }
}

// 2 Re( conj(l0) (M p)_0 + conj(l1) (M p)_1 ) for the generator class GEN.
template <int GEN>
__device__ __forceinline__ double grad_pair(const double* mr, const double* mi, const double2& p0, const double2& p1,
                                            const double2& l0, const double2& l1)
{
    if constexpr (GEN == GEN_X) {  // M = -(i/2) X: Im(conj(l0) p1 + conj(l1) p0)
        return fma(l0.x, p1.y, fma(-l0.y, p1.x, fma(l1.x, p0.y, -l1.y * p0.x)));
    } else if constexpr (GEN == GEN_Y) {  // M = -(i/2) Y = [[0, -1/2], [1/2, 0]]
        return fma(l1.x, p0.x, fma(l1.y, p0.y, fma(-l0.x, p1.x, -l0.y * p1.y)));
    } else if constexpr (GEN == GEN_Z) {  // M = diag(-i/2, i/2)
        return fma(l0.x, p0.y, fma(-l0.y, p0.x, fma(-l1.x, p1.y, l1.y * p1.x)));
    } else if constexpr (GEN == GEN_P1) {  // M = diag(0, i)
        return -2.0 * fma(l1.x, p1.y, -l1.y * p1.x);
    } else {
        double m0x = mr[0] * p0.x - mi[0] * p0.y + mr[1] * p1.x - mi[1] * p1.y;
        double m0y = mr[0] * p0.y + mi[0] * p0.x + mr[1] * p1.y + mi[1] * p1.x;
        double m1x = mr[2] * p0.x - mi[2] * p0.y + mr[3] * p1.x - mi[3] * p1.y;
        double m1y = mr[2] * p0.y + mi[2] * p0.x + mr[3] * p1.y + mi[3] * p1.x;
        return 2.0 * (l0.x * m0x + l0.y * m0y + l1.x * m1x + l1.y * m1y);
    }
}

template <int J, bool CTRL, int GEN, int N>
__device__ __forceinline__ double pairs_grad(const double2 (&x)[N], const double2 (&y)[N], const double* mr,
                                             const double* mi, uint32_t ethr, const uint32_t (&er)[N], uint32_t cmask,
                                             uint32_t cval)
{
    double g = 0;
    bool first = true;  // resolved at compile time when CTRL is false
#pragma unroll
    for (int a = 0; a < N; ++a) {
        if (a & (1 << J)) continue;
        const double v = grad_pair<GEN>(mr, mi, x[a], x[a + (1 << J)], y[a], y[a + (1 << J)]);
        if (CTRL) g += (((ethr | er[a]) & cmask) == cval) ? v : 0.0;  // a select
        else g = first ? v : g + v;
        first = false;
    }
    return g;
}

template <int J, bool CTRL, int N>
__device__ __forceinline__ double op_grad(const double2 (&x)[N], const double2 (&y)[N], int gen, const double* mr,
                                          const double* mi, uint32_t ethr, const uint32_t (&er)[N], uint32_t cmask,
                                          uint32_t cval)
{
    switch (gen) {
    case GEN_X: return pairs_grad<J, CTRL, GEN_X>(x, y, mr, mi, ethr, er, cmask, cval);
    case GEN_Y: return pairs_grad<J, CTRL, GEN_Y>(x, y, mr, mi, ethr, er, cmask, cval);
    case GEN_Z: return pairs_grad<J, CTRL, GEN_Z>(x, y, mr, mi, ethr, er, cmask, cval);
    case GEN_P1: return pairs_grad<J, CTRL, GEN_P1>(x, y, mr, mi, ethr, er, cmask, cval);
    default: return pairs_grad<J, CTRL, GEN_DENSE>(x, y, mr, mi, ethr, er, cmask, cval);
    }
}

// ------------------------------------------------------------------------------ tile helpers
struct TileCtx {
    uint64_t base;   // amplitude index bits outside the tile
    uint64_t dth;    // this thread's deposited qubit bits for the load/store mapping
    uint64_t toff;   // element offset of the thread's register 0: (base | dth) * B + bidx
    int b0, bl;      // first batch slot of the tile, this thread's slot offset
    int bidx;        // batch slot this thread loads: b0 + bl, clamped to the last slot
    bool bvalid;     // b0 + bl < B: only then does the thread store
};

// Load/store mapping: element e = th + r * nthr; the low c bits of th are the batch slot, the
// next t - RB - c bits of th and then the RB bits of r are the tile qubits in ascending order.
// tid: the tile (of a launch over one state: blockIdx.x).
template <int RB, typename A> __device__ __forceinline__ TileCtx tile_ctx(const A& a, int th, uint64_t tid)
{
    TileCtx tc;
    uint64_t base = 0;
#pragma unroll
    for (int j = 0; j < 40; ++j)
        if (j < a.nnt) base |= ((tid >> j) & uint64_t(1)) << a.nontile_qubits[j];
    tc.base = base;
    const int c = a.c, t = a.t;
    uint64_t dth = 0;
    const uint32_t q = (uint32_t)th >> c;
#pragma unroll
    for (int j = 0; j < kMaxTileBits; ++j)
        if (j < t - RB - c) dth |= (uint64_t)((q >> j) & 1u) << a.tile_qubits[j];
    tc.dth = dth;
    tc.b0 = blockIdx.y << c;
    tc.bl = th & ((1 << c) - 1);
    tc.bvalid = tc.b0 + tc.bl < a.B;
    tc.bidx = tc.bvalid ? tc.b0 + tc.bl : a.B - 1;
    tc.toff = (base | dth) * (uint64_t)a.B + (uint64_t)tc.bidx;
    return tc;
}

// LDS tile bits of the thread part (the low nb bits of th) of a stored element.
template <typename A> __device__ __forceinline__ uint32_t store_thread_bits(const A& a, int th, int nb)
{
    uint32_t v = 0;
#pragma unroll
    for (int i = 0; i < kMaxTileBits; ++i)
        if (i < nb) v |= (((uint32_t)th >> i) & 1u) << a.ssrc[i];
    return v;
}

// The register bits of the load mapping are tile qubits whose offsets are the same for every
// thread: the host passes them per register.
template <int RB, typename A> __device__ __forceinline__ uint64_t tile_off(const A& a, const TileCtx& tc, int r)
{
    return tc.toff + a.rofs[r];
}

// Tile index of register element r in a register group, split into the per-thread part
// (ethr) and the per-register part (er[r], the same for every thread).
template <int RB>
__device__ __forceinline__ void group_index(const int (&rpos)[kMaxRegBits], int t, int th, uint32_t& ethr,
                                            uint32_t (&er)[1 << RB])
{
    uint32_t rmask = 0;
#pragma unroll
    for (int j = 0; j < RB; ++j) rmask |= 1u << rpos[j];
    uint32_t v = 0;
    int k = 0;
    for (int b = 0; b < t; ++b) {
        if ((rmask >> b) & 1u) continue;
        v |= (((uint32_t)th >> k) & 1u) << b;
        ++k;
    }
    ethr = v;
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
        uint32_t e = 0;
#pragma unroll
        for (int j = 0; j < RB; ++j) e |= ((uint32_t)(r >> j) & 1u) << rpos[j];
        er[r] = e;
    }
}

// The dense block matrices of a forward pass are copied to LDS in 16-byte words; the first
// kDmRegs words of every thread are loaded together with the tile (one wait for both), with
// indices clamped so that every load is in bounds.
static_assert(sizeof(POp) % 16 == 0 && sizeof(PGroupDesc) % 16 == 0, "16-byte records");
constexpr int kDmRegs = 4;
// With no dense matrices the words are read from the first op record (every forward pass has
// one) and dropped, so the registers are always defined.
template <typename A> __device__ __forceinline__ void dm_load(const A& a, int th, int nthr, uint4 (&w)[kDmRegs])
{
    const uint4* src = a.ndm > 0 ? a.dmats : (const uint4*)a.ops;
    const int last = a.ndm > 0 ? a.ndm - 1 : 0;
#pragma unroll
    for (int k = 0; k < kDmRegs; ++k) w[k] = src[min(th + k * nthr, last)];
}
template <typename A> __device__ __forceinline__ void dm_store(const A& a, uint4* ldm, int th, int nthr, const uint4 (&w)[kDmRegs])
{
    // Unconditional: a clamped index writes the word it loaded, so duplicates are identical.
#pragma unroll
    for (int k = 0; k < kDmRegs; ++k) ldm[min(th + k * nthr, a.ndm - 1)] = w[k];
    for (int i = th + kDmRegs * nthr; i < a.ndm; i += nthr) ldm[i] = a.dmats[i];
}

struct GroupCtl {
    int lds, op0, nops;
    int rpos[kMaxRegBits];
};
__device__ __forceinline__ GroupCtl group_ctl_c(const YAO_CONST PGroupDesc* g)
{
    GroupCtl o;
    o.lds = g->lds;
    o.op0 = g->op0;
    o.nops = g->nops;
#pragma unroll
    for (int j = 0; j < kMaxRegBits; ++j) o.rpos[j] = g->rpos[j];
    return o;
}

// ------------------------------------------------------------------------------ gradient sums
// v from lane (lane op CTRL) of the same DPP row, both 32-bit halves. The patterns used here
// read inside the row only, so every source lane is valid.
template <int CTRL> __device__ __forceinline__ double dpp_f64(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Sum of v over the lanes of a 16-lane row that share this lane's low c bits (its batch slot
// of the tile); lanes 0 .. 2^c - 1 of the row end with the sums of slots 0 .. 2^c - 1. Every
// lane of the row must be active.
__device__ __forceinline__ double row_sum(double v, int c)
{
    if (c < 1) v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]: lane ^ 1
    if (c < 2) v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]: lane ^ 2
    if (c < 3) v += dpp_f64<0x124>(v);  // row_ror 4
    v += dpp_f64<0x128>(v);             // row_ror 8
    return v;
}

// Reduce partials red[s * E + e] for gradient s < S (entry e holds batch slot e mod 2^c) to
// one value per (gradient, batch slot b0 + j of the tile) and store it in gpartial at
// ((slot_of(s) * B + b0 + j) * pstride + col). The order of the sums is fixed.
template <typename SlotOf>
__device__ __forceinline__ void reduce_partials(double* __restrict__ gpartial, int B, int pstride, int c,
                                                const double* red, SlotOf slot_of, int S, int E, int nthr, int th,
                                                int col, int b0)
{
    const int Bc = 1 << c;
    if (nthr >= 16) {
        for (int task = th; task < S * 16; task += nthr) {
            const int s = task >> 4, j = task & 15;
            double v = 0;
            for (int e = j; e < E; e += 16) v += red[s * E + e];
            for (int off = 8; off >= Bc; off >>= 1) v += __shfl_xor(v, off, 16);
            if (j < Bc && b0 + j < B) gpartial[((uint64_t)slot_of(s) * B + b0 + j) * pstride + col] = v;
        }
    } else {
        for (int task = th; task < S * Bc; task += nthr) {
            const int s = task / Bc, bb = task % Bc;
            double v = 0;
            for (int e = bb; e < E; e += Bc) v += red[s * E + e];
            if (b0 + bb < B) gpartial[((uint64_t)slot_of(s) * B + b0 + bb) * pstride + col] = v;
        }
    }
}

// Sorted target positions and member offsets of a K-qubit op inside the tile.
template <int K> struct LdsGeom {
    int sorted[K];
    uint32_t off[1 << K];
};

template <int K> __device__ __forceinline__ LdsGeom<K> lds_geom(const int* tpos)
{
    LdsGeom<K> g;
#pragma unroll
    for (int i = 0; i < K; ++i) g.sorted[i] = tpos[i];
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
        for (int j = i + 1; j < K; ++j)
            if (g.sorted[j] < g.sorted[i]) {
                int tmp = g.sorted[i];
                g.sorted[i] = g.sorted[j];
                g.sorted[j] = tmp;
            }
#pragma unroll
    for (int s = 0; s < (1 << K); ++s) {
        uint32_t o = 0;
#pragma unroll
        for (int j = 0; j < K; ++j)
            if ((s >> j) & 1) o |= 1u << tpos[j];
        g.off[s] = o;
    }
    return g;
}

template <int K> __device__ __forceinline__ uint32_t lds_base(uint32_t gidx, const LdsGeom<K>& g)
{
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const uint32_t lo = gidx & ((1u << g.sorted[i]) - 1);
        gidx = ((gidx >> g.sorted[i]) << (g.sorted[i] + 1)) | lo;
    }
    return gidx;
}

template <typename RP, int K>
__device__ __noinline__ void lds_op_fwd(vec2_t<RP>* lp, const YAO_CONST POp* rec, const double* m, int t, int th,
                                        int nthr)
{
    using VP = vec2_t<RP>;
    constexpr int D = 1 << K, DD = D * D;
    int tpos[K];
#pragma unroll
    for (int j = 0; j < K; ++j) tpos[j] = sc(rec->tpos[j]);
    const uint32_t cmask = (uint32_t)sc((int)rec->cmask), cval = (uint32_t)sc((int)rec->cval);
    const LdsGeom<K> g = lds_geom<K>(tpos);
    for (int gidx = th; gidx < (1 << (t - K)); gidx += nthr) {
        const uint32_t eb = lds_base<K>((uint32_t)gidx, g);
        if ((eb & cmask) != cval) continue;
        VP v[D];
#pragma unroll
        for (int s = 0; s < D; ++s) v[s] = lp[swz(eb | g.off[s])];
#pragma unroll
        for (int r = 0; r < D; ++r) {
            RP x = 0, y = 0;
#pragma unroll
            for (int s = 0; s < D; ++s) {
                const RP ur = (RP)m[r * D + s], ui = (RP)m[DD + r * D + s];
                x = fma(ur, v[s].x, fma(-ui, v[s].y, x));
                y = fma(ur, v[s].y, fma(ui, v[s].x, y));
            }
            lp[swz(eb | g.off[r])] = mkv<VP, RP>(x, y);
        }
    }
}

template <typename RL, int K>
__device__ __noinline__ double lds_op_bwd(double2* lp, vec2_t<RL>* ll, const YAO_CONST POp* rec, const double* m, int t, int th,
                                          int nthr)
{
    using VL = vec2_t<RL>;
    constexpr int D = 1 << K, DD = D * D;
    int tpos[K];
#pragma unroll
    for (int j = 0; j < K; ++j) tpos[j] = sc(rec->tpos[j]);
    const uint32_t cmask = (uint32_t)sc((int)rec->cmask), cval = (uint32_t)sc((int)rec->cval);
    const bool grad = sc(rec->slot) >= 0;
    const LdsGeom<K> g = lds_geom<K>(tpos);
    const double* Mr = m + 2 * DD;
    const double* Mi = m + 3 * DD;
    double acc = 0;
    for (int gidx = th; gidx < (1 << (t - K)); gidx += nthr) {
        const uint32_t eb = lds_base<K>((uint32_t)gidx, g);
        if ((eb & cmask) != cval) continue;
        double2 p[D], l[D];
#pragma unroll
        for (int s = 0; s < D; ++s) {
            p[s] = lp[swz(eb | g.off[s])];
            const VL w = ll[swz(eb | g.off[s])];
            l[s] = make_double2((double)w.x, (double)w.y);
        }
        if (grad) {
#pragma unroll
            for (int r = 0; r < D; ++r) {
                double x = 0, y = 0;
#pragma unroll
                for (int s = 0; s < D; ++s) {
                    x += Mr[r * D + s] * p[s].x - Mi[r * D + s] * p[s].y;
                    y += Mr[r * D + s] * p[s].y + Mi[r * D + s] * p[s].x;
                }
                acc += 2.0 * (l[r].x * x + l[r].y * y);
            }
        }
#pragma unroll
        for (int r = 0; r < D; ++r) {
            double x = 0, y = 0, u = 0, w = 0;
#pragma unroll
            for (int s = 0; s < D; ++s) {
                const double ur = m[r * D + s], ui = m[DD + r * D + s];
                x += ur * p[s].x - ui * p[s].y;
                y += ur * p[s].y + ui * p[s].x;
                u += ur * l[s].x - ui * l[s].y;
                w += ur * l[s].y + ui * l[s].x;
            }
            lp[swz(eb | g.off[r])] = make_double2(x, y);
            ll[swz(eb | g.off[r])] = mkv<VL, RL>((RL)u, (RL)w);
        }
    }
    return acc;
}

// y = M x for the 16 register elements of a thread. M sits in LDS column-major: column c is
// re[16] then im[16] in the precision RR; every lane reads the same address (broadcast).
template <typename RR, typename V>
__device__ __forceinline__ void dense16_apply(V (&x)[16], const RR* M)
{
    RR yr[16], yi[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) yr[r] = yi[r] = (RR)0;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        const RR* col = M + c * 32;
        const RR xr = x[c].x, xi = x[c].y;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const RR mr = col[r], mi = col[16 + r];
            yr[r] = fma(mr, xr, yr[r]);
            yi[r] = fma(mr, xi, yi[r]);
            yr[r] = fma(-mi, xi, yr[r]);
            yi[r] = fma(mi, xr, yi[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = mkv<V, RR>(yr[r], yi[r]);
}

typedef float v4f __attribute__((ext_vector_type(4)));

// A dense block on the FP32 matrix cores, for complex64 tiles of >= 64 columns (one column per
// thread of the group). The block's 4 bits p[0..3] (ascending) index the 16 amplitudes of a
// column; the other t - 4 tile bits number the columns. Taking 16 columns as the B operand
// [Re x; Im x] (32 x 16), the update is the real GEMM [[Re M, -Im M], [Im M, Re M]] x B with
// v_mfma_f32_16x16x4f32 (A[i][k] from lane i + 16 k, B[k][j] from lane j + 16 k,
// D[4 (l / 16) + v][l % 16] in accumulator v of lane l). Each wave takes 64 columns; the
// amplitudes are read from and written back to the LDS tile in that layout, so no barrier
// is needed inside the block. Mf holds the 16 A fragments of 64 lanes each.
__device__ __forceinline__ uint32_t insert_zeros4(uint32_t c, const int (&p)[kMaxRegBits])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) c = ((c >> p[j]) << (p[j] + 1)) | (c & ((1u << p[j]) - 1));
    return c;
}
__device__ __forceinline__ uint32_t deposit4(uint32_t b, const int (&p)[kMaxRegBits])
{
    uint32_t e = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) e |= ((b >> j) & 1u) << p[j];
    return e;
}
__device__ __forceinline__ void dense16_mfma(float2* lp, const float2* M, const int (&p)[kMaxRegBits], int th,
                                             uint32_t cmask, uint32_t cval)
{
    const int lane = th & 63, wave = th >> 6;
    const int q = lane >> 4, cl = lane & 15;
    // A fragments of the real form: row 16 rt + cl, column 4 kc + q, from the complex matrix
    // M (row-major, 16 x 16): Re, -Im in the upper half, Im, Re in the lower one.
    float a[16];
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) {
        const float2 m = M[cl * 16 + 4 * kc + q];
        a[kc] = m.x;
        a[4 + kc] = -m.y;
        a[8 + kc] = m.y;
        a[12 + kc] = m.x;
    }
    uint32_t bin[4], bout[4];
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2) {
        bin[s2] = deposit4((uint32_t)(q + 4 * s2), p);
        bout[s2] = deposit4((uint32_t)(4 * q + s2), p);
    }
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
        const uint32_t ec = insert_zeros4((uint32_t)(wave * 64 + ct * 16 + cl), p);
        float2 xv[4];
#pragma unroll
        for (int s2 = 0; s2 < 4; ++s2) xv[s2] = lp[swz(ec | bin[s2])];
        v4f acc0 = v4f{0.f, 0.f, 0.f, 0.f}, acc1 = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kc = 0; kc < 8; ++kc) {
            const float bv = kc < 4 ? xv[kc].x : xv[kc - 4].y;
            acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kc], bv, acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[8 + kc], bv, acc1, 0, 0, 0);
        }
        if ((ec & cmask) == cval) {
#pragma unroll
            for (int v = 0; v < 4; ++v) lp[swz(ec | bout[v])] = make_float2(acc0[v], acc1[v]);
        }
    }
}

// ------------------------------------------------------------------------------ forward kernel
template <typename RP, typename Args>
__device__ __forceinline__ void pass_fwd(const Args& a, uint64_t tile, unsigned char* smem)
{
    constexpr int RB = kRegBitsFwd, N = 1 << RB;
    using VP = vec2_t<RP>;
    const int t = a.t;
    const int nthr = 1 << (t - RB);
    const int th = threadIdx.x;
    // LDS: tile | dense block matrices (2 * 256 RP each), sized for this pass.
    VP* lp = (VP*)smem;
    uint4* ldm = (uint4*)(smem + (sizeof(VP) << t));
    const YAO_CONST POp* gops = cptr(z_ops(a));
    const YAO_CONST PGroupDesc* ggrp = cptr(a.groups);
    const TileCtx tc = tile_ctx<RB>(a, th, tile);
    VP* gp = (VP*)z_psi(a);
    // Every load is in bounds (slots past B read the last slot and are never stored), so all
    // of them are issued before the first wait.
    {
        uint4 w[kDmRegs];
        dm_load(a, th, nthr, w);
        // The tile goes straight to LDS before the matrices' remaining words: a register copy
        // of it held across that loop stayed in scratch memory.
#pragma unroll
        for (int r = 0; r < N; ++r) lp[swz((uint32_t)th + (uint32_t)r * nthr)] = gp[tile_off<RB>(a, tc, r)];
        if (a.ndm) dm_store(a, ldm, th, nthr, w);
    }
    __syncthreads();

    for (int gi = 0; gi < a.ngroups; ++gi) {
        const GroupCtl G = group_ctl_c(ggrp + gi);
        if (G.lds == 2) {
            // One dense block on the register bits; its remaining controls are on tile bits
            // outside them (the same for all 16 elements of a thread) or outside the tile.
            OpCtl op = op_ctl_c(gops + G.op0);
            fold_outer_controls(op, tc.base);
            if constexpr (sizeof(RP) == 4) {
                // Complex64 plans hold dense blocks only for tiles of >= 64 columns.
                dense16_mfma(lp, (const float2*)ldm + op.mat * 256, G.rpos, th, op.cmask, op.cval);
            } else {
                uint32_t ethr, er[N];
                group_index<RB>(G.rpos, t, th, ethr, er);
                VP x[N];
#pragma unroll
                for (int r = 0; r < N; ++r) x[r] = lp[swz(ethr | er[r])];
                if ((ethr & op.cmask) == op.cval) dense16_apply<RP>(x, (const RP*)ldm + op.mat * 512);
#pragma unroll
                for (int r = 0; r < N; ++r) lp[swz(ethr | er[r])] = x[r];
            }
            __syncthreads();
            continue;
        }
        if (G.lds) {
            const YAO_CONST POp* rec = gops + G.op0;
            const uint64_t omask = rec->omask, oval = rec->oval;
            if ((tc.base & omask) == oval) {
                const double* m = a.mats + rec->mat;
                if (rec->k == 2) lds_op_fwd<RP, 2>(lp, rec, m, t, th, nthr);
                else lds_op_fwd<RP, 3>(lp, rec, m, t, th, nthr);
            }
            __syncthreads();
            continue;
        }
        uint32_t ethr, er[N];
        group_index<RB>(G.rpos, t, th, ethr, er);
        VP x[N];
#pragma unroll
        for (int r = 0; r < N; ++r) x[r] = lp[swz(ethr | er[r])];
        // One op: the common classes (see op_variant: no controls outside the tile, and none
        // at all but for the controlled SWAP) have in-place code of their own, picked by one
        // switch on the variant the host chose; the rest take the masked dense update.
        auto apply = [&](const OpS<RP>& o) __attribute__((always_inline)) {
            const RP* mr = o.m;
            const RP* mi = o.m + 4;
#define YAO_FWD_CASE(J)                                                  \
    case J: {                                                            \
        OpCtl op = o.c;                                                  \
        fold_outer_controls(op, tc.base);                                \
        pairs_dense_ctl_ip<J>(x, mr, mi, ethr, er, op.cmask, op.cval);   \
        break;                                                           \
    }
#define YAO_FWD_FAST(J)                                                                            \
    case 0 * kRegBitsFwd + J: pairs_ip<J, OT_RX>(x, mr, mi); break;                                 \
    case 1 * kRegBitsFwd + J: pairs_ip<J, OT_DIAG>(x, mr, mi); break;                               \
    case 2 * kRegBitsFwd + J: pairs_ip<J, OT_DENSE>(x, mr, mi); break;                              \
    case 3 * kRegBitsFwd + J: pairs_cswap_ip<J>(x, ethr, er, o.c.cmask, o.c.cval); break;
            switch (o.c.var) {
                YAO_FWD_FAST(0) YAO_FWD_FAST(1) YAO_FWD_FAST(2) YAO_FWD_FAST(3)
            default:
                switch (o.c.rpos) { YAO_FWD_CASE(0) YAO_FWD_CASE(1) YAO_FWD_CASE(2) default: YAO_FWD_CASE(3) }
                break;
            }
#undef YAO_FWD_FAST
#undef YAO_FWD_CASE
        };
        // Two record buffers in turn: the record of the next op is loaded (scalar loads) while
        // the current one computes, and is waited for only at the end of it. The record one
        // past a group's last op is always readable (it lies inside the program's buffer) and
        // is never used.
        // Scalar loads return out of order, so each buffer's wait is placed (and fenced from
        // the scheduler) before the other buffer's loads are issued; otherwise it would also
        // wait for the prefetch.
        const YAO_CONST POp* rec = gops + G.op0;
        OpS<RP> A = load_op_c<RP>(rec);
        for (int oi = 0; oi < G.nops; oi += 2) {
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): A (and the LDS reads) arrived
            __builtin_amdgcn_sched_barrier(0);
            const OpS<RP> B = load_op_c<RP>(rec + oi + 1);
            apply(A);
            if (oi + 1 >= G.nops) break;
            __builtin_amdgcn_s_waitcnt(0xC07F);  // B arrived
            __builtin_amdgcn_sched_barrier(0);
            A = load_op_c<RP>(rec + oi + 2);
            apply(B);
        }
#pragma unroll
        for (int r = 0; r < N; ++r) lp[swz(ethr | er[r])] = x[r];
        __syncthreads();
    }

    if (tc.bvalid) {
        const uint32_t sth = store_thread_bits(a, th, t - RB);
#pragma unroll
        for (int r = 0; r < N; ++r) gp[tile_off<RB>(a, tc, r)] = lp[swz(sth | a.sreg[r])];
    }
}

template <typename RP>
__global__ __launch_bounds__(512, sizeof(RP) == 4 ? 3 : 1) void k_pass_fwd(PassArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    pass_fwd<RP>(a, blockIdx.x, smem);
}

// One pass of each of several circuits at once: block b works on tile blocks[b].y of items[blocks[b].x].
template <typename RP>
__global__ __launch_bounds__(512, sizeof(RP) == 4 ? 3 : 1) void k_pass_fwd_many(const PassArgs* items, const uint2* blocks)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const uint2 b = {(uint32_t)sc((int)blocks[blockIdx.x].x), (uint32_t)sc((int)blocks[blockIdx.x].y)};
    pass_fwd<RP>(cptr(items)[b.x], b.y, smem);
}

// ------------------------------------------------------------------------------ backward kernel

// Where the gradient partials of a reverse sweep go: reduce_partials' gpartial, B, pstride
// and, for this tile, the column and the first batch slot.
struct GradOut {
    double* gpartial;
    int B, pstride, col, b0;
};

// The register groups and LDS ops of a reverse pass over the tile in LDS: psi (lp, FP64) and
// lambda (ll, in RL), with every gradient partial reduced per group into go. tbase holds the
// qubits outside the tile (for controls there); red0 holds two buffers of mslots * E
// partials (a group's partials are reduced after the barrier that ends it, while the next
// group fills the other buffer). C0: tiles of one batch slot (c = 0).
template <typename RL, bool C0>
__device__ __forceinline__ double2 reverse_groups(double2* lp, vec2_t<RL>* ll, double* red0, const YAO_CONST POp* gops,
                                               const YAO_CONST PGroupDesc* ggrp, const PGroupDesc* groups,
                                               int ngroups, const double* mats, uint64_t tbase, int t, int c,
                                               int nthr, int th, int mslots, const GradOut& go)
{
    constexpr int RB = kRegBitsBwd, N = 1 << RB;
    using VL = vec2_t<RL>;
    const bool rows = nthr >= 16;
    // Product of the first diagonal entries of the uncontrolled Z-generator ops applied so far:
    // those ops apply diag(1, d1 / d0) to both states and leave d0, a phase common to every
    // element of every tile, to the caller (gradients do not see a phase psi and lambda share).
    double2 phase = make_double2(1.0, 0.0);
    const int E = grad_entries(nthr, c);
    const int ent = rows ? (th >> 4) * (1 << c) + (th & 15) : th;
    const bool stores = rows ? (th & 15) < (1 << c) : true;
    int buf = 0;
    for (int gi = 0; gi < ngroups; ++gi) {
        const GroupCtl G = group_ctl_c(ggrp + gi);
        double* red = red0 + buf * (mslots * E);
        int nslot = 0;
        if (G.lds) {
            const YAO_CONST POp* rec = gops + G.op0;
            const uint64_t omask = rec->omask, oval = rec->oval;
            double g = 0;
            if ((tbase & omask) == oval) {
                const double* m = mats + rec->mat;
                if (rec->k == 2) g = lds_op_bwd<RL, 2>(lp, ll, rec, m, t, th, nthr);
                else g = lds_op_bwd<RL, 3>(lp, ll, rec, m, t, th, nthr);
            }
            if (rec->slot >= 0) {
                if (rows) g = row_sum(g, c);
                if (stores) red[ent] = g;
                nslot = 1;
            }
        } else {
            uint32_t ethr, er[N];
            group_index<RB>(G.rpos, t, th, ethr, er);
            double2 x[N], y[N];
#pragma unroll
            for (int r = 0; r < N; ++r) {
                const uint32_t p = swz(ethr | er[r]);
                x[r] = lp[p];
                const VL w = ll[p];
                y[r] = make_double2((double)w.x, (double)w.y);
            }
            // One op (see the forward kernel): its gradient partial first, from psi and lambda
            // before the update, then U^dagger on both.
            auto apply = [&](const OpS<double>& o) __attribute__((always_inline)) {
                const double* m = o.m;
                double g = 0;
#define YAO_BWD_CASE(J)                                                                                 \
    case J: {                                                                                           \
        OpCtl op = o.c;                                                                                 \
        fold_outer_controls(op, tbase);                                                                 \
        const double* gm = mats + op.mat + 8; /* M of a dense generator */                             \
        if (op.slot >= 0) {                                                                             \
            if (op.cmask) g = op_grad<J, true>(x, y, op.gen, gm, gm + 4, ethr, er, op.cmask, op.cval);  \
            else g = op_grad<J, false>(x, y, op.gen, gm, gm + 4, ethr, er, 0u, 0u);                     \
        }                                                                                               \
        pairs_dense_ctl_ip<J>(x, y, m, m + 4, ethr, er, op.cmask, op.cval);                             \
        break;                                                                                          \
    }
#define YAO_BWD_FAST(J)                                                          \
    case 0 * kRegBitsBwd + J:                                                    \
        g = pairs_grad<J, false, GEN_X>(x, y, m, m + 4, ethr, er, 0u, 0u);         \
        pairs_ip<J, OT_RX>(x, m, m + 4);                                         \
        pairs_ip<J, OT_RX>(y, m, m + 4);                                         \
        break;                                                                   \
    case 1 * kRegBitsBwd + J: {                                                  \
        g = pairs_grad<J, false, GEN_Z>(x, y, m, m + 4, ethr, er, 0u, 0u);         \
        pairs_ip<J, kDiagHigh>(x, m, m + 4);                                     \
        pairs_ip<J, kDiagHigh>(y, m, m + 4);                                     \
        const double pr = phase.x * m[0] - phase.y * m[4];                       \
        phase.y = phase.x * m[4] + phase.y * m[0];                               \
        phase.x = pr;                                                            \
        break;                                                                   \
    }                                                                            \
    case 2 * kRegBitsBwd + J:                                                    \
        pairs_cswap_ip<J>(x, y, ethr, er, o.c.cmask, o.c.cval);                  \
        break;
                switch (o.c.var) {
                    YAO_BWD_FAST(0) YAO_BWD_FAST(1) YAO_BWD_FAST(2)
                default:
                    switch (o.c.rpos) { YAO_BWD_CASE(0) YAO_BWD_CASE(1) default: YAO_BWD_CASE(2) }
                    break;
                }
#undef YAO_BWD_FAST
#undef YAO_BWD_CASE
                if (o.c.slot >= 0) {
                    if (rows) g = row_sum(g, c);
                    if (stores) red[nslot * E + ent] = g;
                    ++nslot;
                }
            };
            // Two record buffers in turn, as in the forward kernel.
            const YAO_CONST POp* rec = gops + G.op0;
            OpS<double> A = load_op_c<double>(rec);
            for (int oi = 0; oi < G.nops; oi += 2) {
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), as in the forward kernel
                __builtin_amdgcn_sched_barrier(0);
                const OpS<double> B = load_op_c<double>(rec + oi + 1);
                apply(A);
                if (oi + 1 >= G.nops) break;
                __builtin_amdgcn_s_waitcnt(0xC07F);
                __builtin_amdgcn_sched_barrier(0);
                A = load_op_c<double>(rec + oi + 2);
                apply(B);
            }
#pragma unroll
            for (int r = 0; r < N; ++r) {
                const uint32_t p = swz(ethr | er[r]);
                lp[p] = x[r];
                ll[p] = mkv<VL, RL>((RL)y[r].x, (RL)y[r].y);
            }
        }
        __syncthreads();
        if (nslot > 0) {
            const int* slots = groups[gi].slots;
            reduce_partials(go.gpartial, go.B, go.pstride, c, red, [&](int s) { return slots[s]; }, nslot, E, nthr,
                            th, go.col, go.b0);
            buf ^= 1;
        }
    }
    return phase;
}

// C0: tiles of one batch slot (c = 0), where every row-sum step applies. At most 168 VGPRs, so
// that three 256-thread tiles of 2^11 elements (48 KiB of LDS each) fit on one CU.
template <typename RL, bool C0, typename Args>
__device__ __forceinline__ void pass_bwd(const Args& a, uint64_t tile, unsigned char* smem)
{
    constexpr int RB = kRegBitsBwd, N = 1 << RB;
    using VL = vec2_t<RL>;
    const int t = a.t;
    const int nthr = 1 << (t - RB);
    const int th = threadIdx.x;
    const int c = C0 ? 0 : a.c;
    // LDS: psi | lambda | gradient partials.
    double2* lp = (double2*)smem;
    VL* ll = (VL*)(smem + ((size_t)16 << t));
    double* red0 = (double*)(smem + ((size_t)(16 + sizeof(VL)) << t));
    const TileCtx tc = tile_ctx<RB>(a, th, tile);
    double2* gp = (double2*)z_psi(a);
    VL* gl = (VL*)z_lam(a);
    // Straight from global memory to LDS: a staging array here stayed in scratch memory
    // (a store and a reload per element through the cache hierarchy).
#pragma unroll
    for (int r = 0; r < N; ++r) {
        const uint64_t off = tile_off<RB>(a, tc, r);
        const uint32_t e = swz((uint32_t)th + (uint32_t)r * nthr);
        lp[e] = gp[off];
        ll[e] = gl[off];
    }
    __syncthreads();

    const GradOut go{z_partial(a, a.gpartial), a.B, a.pstride, (int)tile, (int)blockIdx.y << c};
    const double2 ph = reverse_groups<RL, C0>(lp, ll, red0, cptr(z_ops(a)), cptr(a.groups), a.groups, a.ngroups,
                                              a.mats, tc.base, t, c, nthr, th, a.mslots, go);

    if (tc.bvalid) {
        const uint32_t sth = store_thread_bits(a, th, t - RB);
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const uint64_t off = tile_off<RB>(a, tc, r);
            const uint32_t e = swz(sth | a.sreg[r]);
            const double2 v = lp[e];
            const VL w = ll[e];
            const double wx = (double)w.x, wy = (double)w.y;
            gp[off] = make_double2(ph.x * v.x - ph.y * v.y, ph.x * v.y + ph.y * v.x);
            gl[off] = mkv<VL, RL>((RL)(ph.x * wx - ph.y * wy), (RL)(ph.x * wy + ph.y * wx));
        }
    }
}

template <typename RL, bool C0>
__global__ __launch_bounds__(512, 3) void k_pass_bwd(PassArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    pass_bwd<RL, C0>(a, blockIdx.x, smem);
}

// As k_pass_fwd_many, for reverse passes of single-slot states.
template <typename RL>
__global__ __launch_bounds__(512, 3) void k_pass_bwd_many(const PassArgs* items, const uint2* blocks)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const uint2 b = {(uint32_t)sc((int)blocks[blockIdx.x].x), (uint32_t)sc((int)blocks[blockIdx.x].y)};
    pass_bwd<RL, true>(cptr(items)[b.x], b.y, smem);
}

// ------------------------------------------------------------------------------ small circuits
// The register groups and LDS ops of a forward pass with 3 register bits and FP64 matrices
// over a tile in LDS that holds every qubit (no controls outside it, no dense blocks).
__device__ __forceinline__ void forward_groups3(double2* lp, const YAO_CONST POp* gops,
                                                const YAO_CONST PGroupDesc* ggrp, int ngroups, const double* mats,
                                                int t, int nthr, int th)
{
    constexpr int RB = 3, N = 1 << RB;
    for (int gi = 0; gi < ngroups; ++gi) {
        const GroupCtl G = group_ctl_c(ggrp + gi);
        if (G.lds) {
            const YAO_CONST POp* rec = gops + G.op0;
            const double* m = mats + rec->mat;
            if (rec->k == 2) lds_op_fwd<double, 2>(lp, rec, m, t, th, nthr);
            else lds_op_fwd<double, 3>(lp, rec, m, t, th, nthr);
            __syncthreads();
            continue;
        }
        uint32_t ethr, er[N];
        group_index<RB>(G.rpos, t, th, ethr, er);
        double2 x[N];
#pragma unroll
        for (int r = 0; r < N; ++r) x[r] = lp[swz(ethr | er[r])];
        // The forward classes of op_variant on 3 register bits (see the forward kernel).
        auto apply = [&](const OpS<double>& o) __attribute__((always_inline)) {
            const double* mr = o.m;
            const double* mi = o.m + 4;
#define YAO_SF_CASE(J) \
    case J: pairs_dense_ctl_ip<J>(x, mr, mi, ethr, er, o.c.cmask, o.c.cval); break;
#define YAO_SF_FAST(J)                                                               \
    case 0 * RB + J: pairs_ip<J, OT_RX>(x, mr, mi); break;                           \
    case 1 * RB + J: pairs_ip<J, OT_DIAG>(x, mr, mi); break;                         \
    case 2 * RB + J: pairs_ip<J, OT_DENSE>(x, mr, mi); break;                        \
    case 3 * RB + J: pairs_cswap_ip<J>(x, ethr, er, o.c.cmask, o.c.cval); break;
            switch (o.c.var) {
                YAO_SF_FAST(0) YAO_SF_FAST(1) YAO_SF_FAST(2)
            default:
                switch (o.c.rpos) { YAO_SF_CASE(0) YAO_SF_CASE(1) default: YAO_SF_CASE(2) }
                break;
            }
#undef YAO_SF_FAST
#undef YAO_SF_CASE
        };
        const YAO_CONST POp* rec = gops + G.op0;
        OpS<double> A = load_op_c<double>(rec);
        for (int oi = 0; oi < G.nops; oi += 2) {
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), as in the forward kernel
            __builtin_amdgcn_sched_barrier(0);
            const OpS<double> B = load_op_c<double>(rec + oi + 1);
            apply(A);
            if (oi + 1 >= G.nops) break;
            __builtin_amdgcn_s_waitcnt(0xC07F);
            __builtin_amdgcn_sched_barrier(0);
            A = load_op_c<double>(rec + oi + 2);
            apply(B);
        }
#pragma unroll
        for (int r = 0; r < N; ++r) lp[swz(ethr | er[r])] = x[r];
        __syncthreads();
    }
}

// One workgroup per circuit of a batch whose state fits one tile (eq. apply-back and the
// outer-product gradient as in the reverse passes, all in LDS): psi = |0..0>, the forward
// program, psi_N to the state, lambda = H psi and the energy, then the reverse program with
// its gradients. LDS: psi (FP64) | lambda (FP64) | gradient partials.
__global__ __launch_bounds__(512, 1) void k_small_circuit(const SmallCircuit* items)
{
    constexpr int RB = 3, N = 1 << RB;
    extern __shared__ __align__(16) unsigned char smem[];
    const YAO_CONST SmallCircuit* it = cptr(items) + blockIdx.x;
    const int t = it->n;
    const int nthr = 1 << (t - RB);
    const int th = threadIdx.x;
    double2* lp = (double2*)smem;
    double2* ll = lp + (size_t(1) << t);
    double* red0 = (double*)(ll + (size_t(1) << t));
#pragma unroll
    for (int r = 0; r < N; ++r) {
        const uint32_t e = (uint32_t)th + (uint32_t)r * nthr;
        lp[swz(e)] = make_double2(e == 0 ? 1.0 : 0.0, 0.0);
    }
    __syncthreads();
    forward_groups3(lp, cptr(it->fops), cptr(it->fgroups), it->nfg, it->fmats, t, nthr, th);

    // Tile element e is basis state e (the tile holds qubits 0 .. n-1 in order).
    const YAO_CONST PGroup* hg = cptr(it->hgroups);
    const YAO_CONST PTerm* ht = cptr(it->hterms);
    const int nhg = it->nhg;
    const bool c64 = it->c64 != 0;
    double acc = 0;
#pragma unroll
    for (int r = 0; r < N; ++r) {
        const uint32_t e = (uint32_t)th + (uint32_t)r * nthr;
        const double2 a = lp[swz(e)];
        if (c64) ((float2*)it->state)[e] = make_float2((float)a.x, (float)a.y);
        else ((double2*)it->state)[e] = a;
        double orr = 0, oi = 0;
        for (int g = 0; g < nhg; ++g) {
            const uint32_t src = e ^ (uint32_t)hg[g].x;
            const double2 p = lp[swz(src)];
            double cr = 0, ci = 0;  // sum of c i^ny (-1)^{|src & z|}
            for (int k = hg[g].t0; k < hg[g].t1; ++k) {
                const double cc = (__popcll((uint64_t)src & ht[k].z) & 1) ? -ht[k].c : ht[k].c;
                switch (ht[k].ny & 3) {
                case 0: cr += cc; break;
                case 1: ci += cc; break;
                case 2: cr -= cc; break;
                default: ci -= cc; break;
                }
            }
            orr += cr * p.x - ci * p.y;
            oi += cr * p.y + ci * p.x;
        }
        ll[swz(e)] = make_double2(orr, oi);
        acc += a.x * orr + a.y * oi;
    }
    red0[th] = acc;
    __syncthreads();
    if (th == 0) {
        double sum = 0;
        for (int i = 0; i < nthr; ++i) sum += red0[i];
        *it->energy = sum;
    }
    __syncthreads();
    const GradOut go{it->grad, 1, 1, 0, 0};
    reverse_groups<double, true>(lp, ll, red0, cptr(it->rops), cptr(it->rgroups), it->rgroups, it->nrg, it->rmats, 0,
                                 t, 0, nthr, th, kMaxGroupSlots, go);
}

size_t small_circuit_lds_bytes(int n)
{
    const int nthr = 1 << (n - 3);
    return ((size_t)32 << n) + sizeof(double) * 2 * kMaxGroupSlots * (size_t)grad_entries(nthr, 0);
}

// ------------------------------------------------------------------------------ observables
// H psi and <psi|H|psi>: the terms of one X mask x add c_t i^{ny} (-1)^{|(j ^ x) & z|} psi[j ^ x]
// to element j (eq. expectation). A thread holds 2^RB elements that differ in the top RB index
// bits (of its tile, or of the register), so per term it takes one sign, the parity of its own
// index bits, and the signs of its elements relative to each other are the term's class: z's top
// bits. The host folds i^{ny}, |x & z| and the coefficient into one number, puts the terms of a
// mask in order of class, and terms of one class are summed (one FP64 add each) before they meet
// the amplitudes. What bounds it is the vector units: per X mask and amplitude one read of the
// partner and two FMAs per class, per term about one instruction per amplitude (before, six, and
// two FMAs for every term). The 25-qubit Heisenberg energy at complex64 (75 terms, 3 passes) went
// from 295 to about 145 us a pass; reading the partners one mask ahead also in the tile passes took
// 134 VGPRs at complex128 and was slower (24 qubits: 562 against 317 us).
constexpr int kObsRegBits = 3;  // elements per thread: 8
constexpr int kObsMaxTile = 12;
// One term. flags: bits 0..2 class (z on the thread's register bits), bit 3 imaginary (odd ny),
// bit 4 last term of its class within its X mask, bit 5 first term of its X mask.
struct ObsRec {
    double c;
    uint64_t zout;    // Z mask on qubits outside the tile (index coordinates)
    uint32_t zin;     // Z mask on the thread's own bits (tile bits, or the register's low bits)
    uint32_t x;       // X mask (tile bits, or index bits)
    uint32_t xnext;   // X mask of the next one in the list (the last one: 0)
    uint32_t flags;
};
static_assert(sizeof(ObsRec) == 32, "one scalar load");
constexpr uint32_t kObsLast = 16, kObsFirst = 32;

// orr + i oi += f p with f = s (real) or i s (imaginary), for the elements of class CLS: the
// elements whose register bits have odd overlap with CLS take -s.
template <int RB, int CLS, bool IMAG>
__device__ __forceinline__ void obs_add(double s, const double2 (&p)[1 << RB], double (&orr)[1 << RB],
                                        double (&oi)[1 << RB])
{
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
        const double f = (__builtin_popcount(r & CLS) & 1) ? -s : s;
        if constexpr (IMAG) {
            orr[r] = fma(-f, p[r].y, orr[r]);
            oi[r] = fma(f, p[r].x, oi[r]);
        } else {
            orr[r] = fma(f, p[r].x, orr[r]);
            oi[r] = fma(f, p[r].y, oi[r]);
        }
    }
}

// The records rq[0 .. nrec) (one more is readable) over a thread's elements: ethr holds the
// thread's own index bits, base the index bits outside the tile, and fetch(x, q) reads the
// partners of the 2^RB elements under mask x. Records come a step ahead through the scalar cache
// and the partners of the next X mask are read while the current one is worked on.
template <int RB, bool AHEAD, typename V, typename F>
__device__ __forceinline__ void obs_terms(const YAO_CONST ObsRec* rq, int nrec, uint32_t ethr, uint64_t base, F fetch,
                                          double (&orr)[1 << RB], double (&oi)[1 << RB])
{
    constexpr int N = 1 << RB;
#pragma unroll
    for (int r = 0; r < N; ++r) orr[r] = oi[r] = 0;
    V q[N];
    double2 p[N];
    auto load = [&](int k) __attribute__((always_inline)) {
        ObsRec o;
        o.c = rq[k].c;
        o.zout = rq[k].zout;
        o.zin = rq[k].zin;
        o.x = rq[k].x;
        o.xnext = rq[k].xnext;
        o.flags = rq[k].flags;
        return o;
    };
    ObsRec cur = load(0);
    if constexpr (AHEAD) fetch(cur.x, q);
    double s = 0;
    for (int k = 0; k < nrec; ++k) {
        const ObsRec next = load(k + 1);
        if (cur.flags & kObsFirst) {
            if constexpr (!AHEAD) fetch(cur.x, q);
#pragma unroll
            for (int r = 0; r < N; ++r) p[r] = make_double2((double)q[r].x, (double)q[r].y);
            if constexpr (AHEAD) fetch(cur.xnext, q);
        }
        const double cb = (__popcll(base & cur.zout) & 1) ? -cur.c : cur.c;
        const uint64_t sign = (uint64_t)((uint32_t)__popc(ethr & cur.zin) << 31) << 32;
        s += __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, cb) ^ sign);
        if (cur.flags & kObsLast) {
#define YAO_OBS_CASE(C)                                        \
    case C: obs_add<RB, C, false>(s, p, orr, oi); break;       \
    case 8 + C: obs_add<RB, C, true>(s, p, orr, oi); break;
            if constexpr (RB == 3) {
                switch (cur.flags & 15) {
                    YAO_OBS_CASE(0) YAO_OBS_CASE(1) YAO_OBS_CASE(2) YAO_OBS_CASE(3)
                    YAO_OBS_CASE(4) YAO_OBS_CASE(5) YAO_OBS_CASE(6) YAO_OBS_CASE(7)
                }
            } else if constexpr (RB == 1) {
                switch (cur.flags & 15) { YAO_OBS_CASE(0) YAO_OBS_CASE(1) }
            } else {
                static_assert(RB == 2, "1 to 3 register bits");
                switch (cur.flags & 15) { YAO_OBS_CASE(0) YAO_OBS_CASE(1) YAO_OBS_CASE(2) YAO_OBS_CASE(3) }
            }
#undef YAO_OBS_CASE
            s = 0;
        }
        cur = next;
    }
}

// One pass over tiles: a pass reads each tile of psi into LDS once and adds the X masks that lie
// inside the tile's qubits, so the state is read once per pass instead of once per mask. With
// OUT, (H psi) of these masks is written to a.lam (accumulate: added to what earlier passes wrote
// there). The pass's part of <psi|H|psi> per batch slot and tile goes to
// partial[b * W + pcol0 + tile].
template <typename RP, typename RO, bool OUT>
__global__ __launch_bounds__(512) void k_obs_pass(PassArgs a, const ObsRec* __restrict__ recs, int nrec, int accumulate,
                                                  double* __restrict__ partial, int pcol0, int W)
{
    constexpr int RB = kObsRegBits, N = 1 << RB;
    using VP = vec2_t<RP>;
    using VO = vec2_t<RO>;
    extern __shared__ __align__(16) unsigned char smem[];
    const int t = a.t, c = a.c;
    const int nthr = 1 << (t - RB);
    const int th = threadIdx.x;
    VP* lp = (VP*)smem;
    double* red = (double*)(smem + (sizeof(VP) << t));
    const TileCtx tc = tile_ctx<RB>(a, th, blockIdx.x);
    const VP* gp = (const VP*)z_psi(a);
    // Straight from global memory to LDS (a staging array stayed in scratch memory).
#pragma unroll
    for (int r = 0; r < N; ++r) lp[swz((uint32_t)th + (uint32_t)r * nthr)] = gp[tile_off<RB>(a, tc, r)];
    __syncthreads();
    VO* go = (VO*)z_lam(a);
    partial = z_partial(a, partial);
    const uint32_t sw = swz((uint32_t)th);
    uint32_t sr[N];  // the swizzle is linear over XOR
#pragma unroll
    for (int r = 0; r < N; ++r) sr[r] = swz((uint32_t)r * nthr);
    double orr[N], oi[N];
    obs_terms<RB, false, VP>(cptr(recs), nrec, (uint32_t)th, tc.base,
                      [&](uint32_t x, VP (&q)[N]) __attribute__((always_inline)) {
                          const uint32_t sx = sw ^ swz(x);
#pragma unroll
                          for (int r = 0; r < N; ++r) q[r] = lp[sx ^ sr[r]];
                      },
                      orr, oi);
    double acc = 0;
#pragma unroll
    for (int r = 0; r < N; ++r) {
        const VP ae = lp[sw ^ sr[r]];
        acc += (double)ae.x * orr[r] + (double)ae.y * oi[r];
        if constexpr (OUT) {
            if (tc.bvalid) {
                const uint64_t off = tile_off<RB>(a, tc, r);
                double wr = orr[r], wi = oi[r];
                if (accumulate) {
                    const VO prev = go[off];
                    wr += (double)prev.x;
                    wi += (double)prev.y;
                }
                go[off] = mkv<VO, RO>((RO)wr, (RO)wi);
            }
        }
    }
    // Per batch slot of the tile: row sums, then the rows in order.
    const int Bc = 1 << c;
    const int E = grad_entries(nthr, c);
    if (nthr >= 16) {
        acc = row_sum(acc, c);
        if ((th & 15) < Bc) red[(th >> 4) * Bc + (th & 15)] = acc;
    } else {
        red[th] = acc;
    }
    __syncthreads();
    if (th < Bc) {
        double sum = 0;
        for (int k = th; k < E; k += Bc) sum += red[k];
        const int b = (int)(blockIdx.y << c) + th;
        if (b < a.B) partial[(uint64_t)b * W + pcol0 + blockIdx.x] = sum;
    }
}

// The whole observable in one launch for single-slot states (obs_gathers says which): a thread's
// partners are read from global memory (a wave's partners are one or a few contiguous runs for
// any mask). Tiles of 2^12 leave most CUs idle on small states (16 tiles at 16 qubits), where the launch
// is bound by the latency of a handful of dependent steps; on large ones by the reads of the caches.
constexpr int kObsGatherThreads = 256;
template <typename RP, typename RO, bool OUT, int RB>
__device__ __forceinline__ void obs_gather(const vec2_t<RP>* __restrict__ gp, vec2_t<RO>* __restrict__ go, int n,
                                           uint32_t block, const ObsRec* recs, int nrec, double* __restrict__ partial,
                                           double2* __restrict__ psi64, double* red)
{
    constexpr int N = 1 << RB;
    using VP = vec2_t<RP>;
    using VO = vec2_t<RO>;
    const int th = threadIdx.x;
    const uint32_t gid = block * blockDim.x + (uint32_t)th;
    const int top = n - RB;
    VP own[N];
#pragma unroll
    for (int r = 0; r < N; ++r) own[r] = gp[gid | ((uint32_t)r << top)];
    if (psi64) {  // the state widened, for the reverse sweep that starts from H psi
#pragma unroll
        for (int r = 0; r < N; ++r)
            psi64[gid | ((uint32_t)r << top)] = make_double2((double)own[r].x, (double)own[r].y);
    }
    double orr[N], oi[N];
    obs_terms<RB, true, VP>(cptr(recs), nrec, gid, 0,
                      [&](uint32_t x, VP (&q)[N]) __attribute__((always_inline)) {
#pragma unroll
                          for (int r = 0; r < N; ++r) q[r] = gp[(gid ^ x) ^ ((uint32_t)r << top)];
                      },
                      orr, oi);
    double acc = 0;
#pragma unroll
    for (int r = 0; r < N; ++r) {
        acc += (double)own[r].x * orr[r] + (double)own[r].y * oi[r];
        if constexpr (OUT) go[gid | ((uint32_t)r << top)] = mkv<VO, RO>((RO)orr[r], (RO)oi[r]);
    }
    red[th] = acc;
    __syncthreads();
    if (th < 64) {  // every thread of the first wave, in a fixed order
        double v = 0;
        for (int i = th; i < (int)blockDim.x; i += 64) v += red[i];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (th == 0) partial[block] = v;
    }
}

template <typename RP, typename RO, bool OUT, int RB>
__global__ __launch_bounds__(kObsGatherThreads) void k_obs_gather(PassArgs a, const ObsRec* __restrict__ recs, int nrec,
                                                                  double* __restrict__ partial,
                                                                  double2* __restrict__ psi64)
{
    __shared__ double red[kObsGatherThreads];
    obs_gather<RP, RO, OUT, RB>((const vec2_t<RP>*)z_psi(a), (vec2_t<RO>*)z_lam(a), a.n, blockIdx.x, recs, nrec,
                                z_partial(a, partial), psi64, red);
}

// H psi of several states at once: block b is block blocks[b].y of items[blocks[b].x].
template <typename R, int RB>
__global__ __launch_bounds__(kObsGatherThreads) void k_obs_gather_many(const ManyObs* items, const uint2* blocks)
{
    __shared__ double red[kObsGatherThreads];
    const uint32_t x = (uint32_t)sc((int)blocks[blockIdx.x].x), y = (uint32_t)sc((int)blocks[blockIdx.x].y);
    const YAO_CONST ManyObs* it = cptr(items) + x;
    obs_gather<R, R, true, RB>((const vec2_t<R>*)it->psi, (vec2_t<R>*)it->lam, it->n, y, (const ObsRec*)it->recs, it->nrec,
                               it->partial, (double2*)it->psi64, red);
}

// Row sums of several blocks of partials at once (a wave a row), and |0...0> into several states.
__global__ __launch_bounds__(256) void k_rows_many(const ManyRows* items, const uint2* blocks)
{
    const uint32_t x = (uint32_t)sc((int)blocks[blockIdx.x].x), y = (uint32_t)sc((int)blocks[blockIdx.x].y);
    const YAO_CONST ManyRows* it = cptr(items) + x;
    const int lane = threadIdx.x & 63, r = (int)y * 4 + (int)(threadIdx.x >> 6);
    if (r >= it->rows) return;
    const double* row = it->partial + (uint64_t)r * it->W;
    double v = 0;
    for (int j = lane; j < it->W; j += 64) v += row[j];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if (lane == 0) it->out[r] = v;
}
template <typename R> __global__ __launch_bounds__(256) void k_reset_many(void* const* states, const int* n)
{
    vec2_t<R>* s = (vec2_t<R>*)states[blockIdx.y];
    const uint64_t elems = uint64_t(1) << n[blockIdx.y];
    for (uint64_t e = (uint64_t)blockIdx.x * 256 + threadIdx.x; e < elems; e += (uint64_t)gridDim.x * 256)
        s[e] = mkv<vec2_t<R>, R>(e == 0 ? R(1) : R(0), R(0));
}

// A step of the Lanczos recurrence as one launch: v = src / |src|, out = H v and the partials of
// <v|H v>, where |src|^2 comes as the nn partials that the step before left. Every workgroup adds them up
// for itself, in one order, so no launch stands between; workgroup 0 leaves |src| in *norm. The
// partners' values are divided as they are read (src and out are different buffers). A vanished src
// gives v = 0 (the Krylov space closed).
template <typename R, int RB>
__global__ __launch_bounds__(kObsGatherThreads) void k_lanczos_hv(const vec2_t<R>* __restrict__ src,
                                                                  vec2_t<R>* __restrict__ v, vec2_t<R>* __restrict__ out,
                                                                  int n, const ObsRec* __restrict__ recs, int nrec,
                                                                  const double* __restrict__ npart, int nn,
                                                                  double* __restrict__ norm, double* __restrict__ partial)
{
    constexpr int N = 1 << RB;
    using V = vec2_t<R>;
    __shared__ double red[kObsGatherThreads];
    const int th = threadIdx.x;
    const uint32_t gid = blockIdx.x * blockDim.x + (uint32_t)th;
    const int top = n - RB;
    V own[N];
#pragma unroll
    for (int r = 0; r < N; ++r) own[r] = src[gid | ((uint32_t)r << top)];
    const double nrm = sqrt(block_total(npart, nn, red));
    if (gid == 0) *norm = nrm;
    const R inv = nrm > 1e-300 ? (R)(1.0 / nrm) : R(0);
#pragma unroll
    for (int r = 0; r < N; ++r) {
        own[r].x *= inv;
        own[r].y *= inv;
        v[gid | ((uint32_t)r << top)] = own[r];
    }
    double orr[N], oi[N];
    obs_terms<RB, true, V>(cptr(recs), nrec, gid, 0,
                           [&](uint32_t x, V (&q)[N]) __attribute__((always_inline)) {
#pragma unroll
                               for (int r = 0; r < N; ++r) {
                                   q[r] = src[(gid ^ x) ^ ((uint32_t)r << top)];
                                   q[r].x *= inv;
                                   q[r].y *= inv;
                               }
                           },
                           orr, oi);
    double acc = 0;
#pragma unroll
    for (int r = 0; r < N; ++r) {
        acc += (double)own[r].x * orr[r] + (double)own[r].y * oi[r];
        out[gid | ((uint32_t)r << top)] = mkv<V, R>((R)orr[r], (R)oi[r]);
    }
    red[th] = acc;
    __syncthreads();
    if (th < 64) {
        double t = 0;
        for (int i = th; i < (int)blockDim.x; i += 64) t += red[i];
        for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
        if (th == 0) partial[blockIdx.x] = t;
    }
}

// Raise each pass kernel's dynamic LDS limit to the CU's 160 KiB, once per kernel.
template <typename K> int set_lds_limit(K kernel)
{
    static std::mutex mu;
    static std::vector<const void*> done;
    std::lock_guard<std::mutex> lk(mu);
    for (const void* k : done)
        if (k == (const void*)kernel) return 0;
    YAO_HIP(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    done.push_back((const void*)kernel);
    return 0;
}

// One-qubit matrix of a gate kind at angle th: rotations exp(-i th S / 2), shift(th) =
// diag(1, e^{i th}), and the fixed Pauli, Hadamard, S and T gates (the same definitions as the
// host's gate matrices).
__device__ void gate2(int kind, double th, double (&r)[4], double (&i)[4])
{
    const double h = 0.70710678118654752440;
    for (int e = 0; e < 4; ++e) r[e] = i[e] = 0.0;
    double sn, cs;
    switch (kind) {
    case YAO_X: r[1] = r[2] = 1.0; break;
    case YAO_Y: i[1] = -1.0; i[2] = 1.0; break;
    case YAO_Z: r[0] = 1.0; r[3] = -1.0; break;
    case YAO_H: r[0] = r[1] = r[2] = h; r[3] = -h; break;
    case YAO_S: r[0] = 1.0; i[3] = 1.0; break;
    case YAO_SDAG: r[0] = 1.0; i[3] = -1.0; break;
    case YAO_T: r[0] = 1.0; r[3] = h; i[3] = h; break;
    case YAO_TDAG: r[0] = 1.0; r[3] = h; i[3] = -h; break;
    case YAO_SHIFT: sincos(th, &sn, &cs); r[0] = 1.0; r[3] = cs; i[3] = sn; break;
    case YAO_RX: sincos(0.5 * th, &sn, &cs); r[0] = r[3] = cs; i[1] = i[2] = -sn; break;
    case YAO_RY: sincos(0.5 * th, &sn, &cs); r[0] = r[3] = cs; r[1] = -sn; r[2] = sn; break;
    case YAO_RZ: sincos(0.5 * th, &sn, &cs); r[0] = r[3] = cs; i[0] = -sn; i[3] = sn; break;
    default: r[0] = r[3] = 1.0; break;
    }
}

// Parameter binding: one thread per bound record multiplies its factors (in application
// order) and writes the matrix into the record (see BindRec).
// The matrix of one bound record: the product of its factors (gate kind and angle), written
// as U (forward, float or double) or U^dagger (reverse) into the record.
__device__ void bind_one(POp* __restrict__ ops, const BindRec br, const BindFac* __restrict__ facs,
                         const double* __restrict__ params)
{
    double ar[4] = {1.0, 0.0, 0.0, 1.0}, ai[4] = {0.0, 0.0, 0.0, 0.0};
    for (int f = 0; f < br.nf; ++f) {
        const BindFac x = facs[br.f0 + f];
        double gr[4], gi[4];
        gate2(x.kind, x.param >= 0 ? params[x.param] : x.theta, gr, gi);
        double nr[4], ni[4];
        for (int row = 0; row < 2; ++row)
            for (int col = 0; col < 2; ++col) {
                const int o = 2 * row + col;
                nr[o] = gr[2 * row] * ar[col] - gi[2 * row] * ai[col] + gr[2 * row + 1] * ar[2 + col] -
                        gi[2 * row + 1] * ai[2 + col];
                ni[o] = gr[2 * row] * ai[col] + gi[2 * row] * ar[col] + gr[2 * row + 1] * ai[2 + col] +
                        gi[2 * row + 1] * ar[2 + col];
            }
        for (int e = 0; e < 4; ++e) {
            ar[e] = nr[e];
            ai[e] = ni[e];
        }
    }
    if (br.mode >= 2 && br.mode <= 4) {  // U^dagger
        double t = ar[1];
        ar[1] = ar[2];
        ar[2] = t;
        t = ai[1];
        ai[1] = -ai[2];
        ai[2] = -t;
        ai[0] = -ai[0];
        ai[3] = -ai[3];
    }
    POp& op = ops[br.op];
    if (br.mode == 5) {
        real_form(ar, ai, (float*)op.u);
        return;
    }
    if (br.mode == 0) {
        float* u = (float*)op.u;
        for (int e = 0; e < 4; ++e) {
            u[e] = (float)ar[e];
            u[4 + e] = (float)ai[e];
        }
    } else {
        for (int e = 0; e < 4; ++e) {
            op.u[e] = ar[e];
            op.u[4 + e] = ai[e];
        }
        if (br.mode == 3) {
            split_rotation(op.u, op.u[4]);
            split_diag_phase(op.u);
        }
        if (br.mode == 4) split_rotation(op.u, op.u[5]);
    }
}

__global__ void k_bind(POp* __restrict__ ops, const BindRec* __restrict__ binds, int nb,
                       const BindFac* __restrict__ facs, const double* __restrict__ params)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nb) return;
    bind_one(ops, binds[b], facs, params);
}

// Two programs for one set of parameters (a step's forward and reverse sweep), and a copy (its input).
__global__ void k_bind_pair(BindJob a, BindJob b, CopyJob copy)
{
    if (blockIdx.y == 2) {
        for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < copy.count; e += (uint64_t)gridDim.x * blockDim.x)
            copy.dst[e] = copy.src[e];
        return;
    }
    const BindJob& j = blockIdx.y ? b : a;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= j.nb) return;
    bind_one(j.ops, j.binds[k], j.facs, j.params);
}

// Many programs at once: job blockIdx.y, record blockIdx.x * blockDim.x + threadIdx.x.
__global__ void k_bind_jobs(const BindJob* __restrict__ jobs)
{
    const BindJob j = jobs[blockIdx.y];
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= j.nb) return;
    bind_one(j.ops, j.binds[b], j.facs, j.params);
}

}  // namespace

int launch_bind_jobs(const BindJob* jobs, int njobs, int max_nb)
{
    if (njobs <= 0 || max_nb <= 0) return 0;
    for (int j = 0; j < njobs; j += 65535) {
        k_bind_jobs<<<dim3((max_nb + 255) / 256, std::min(njobs - j, 65535)), 256, 0, stream()>>>(jobs + j);
        YAO_HIP(hipGetLastError());
    }
    return 0;
}

int launch_small_circuits(const SmallCircuit* items, int count, int n)
{
    if (count <= 0) return 0;
    if (n < 5 || n > kSmallMaxQubits) return set_error(YAO_EINVAL, "small-circuit kernel takes 5..%d qubits, not %d",
                                                       kSmallMaxQubits, n);
    YAO_TRY(set_lds_limit(k_small_circuit));
    k_small_circuit<<<count, 1 << (n - 3), small_circuit_lds_bytes(n), stream()>>>(items);
    YAO_HIP(hipGetLastError());
    return 0;
}

int launch_bind(POp* ops, const BindRec* binds, int nbinds, const BindFac* facs, const double* params)
{
    if (nbinds <= 0) return 0;
    k_bind<<<(nbinds + 255) / 256, 256, 0, stream()>>>(ops, binds, nbinds, facs, params);
    YAO_HIP(hipGetLastError());
    return 0;
}

int launch_bind_pair(const BindJob& a, const BindJob& b, const CopyJob& copy)
{
    const int nb = std::max(a.nb, b.nb);
    if (nb <= 0 && copy.count == 0) return 0;
    const int gx = std::max((nb + 255) / 256, (int)std::min<uint64_t>((copy.count + 255) / 256, 1024));
    k_bind_pair<<<dim3(gx, copy.count ? 3 : 2), 256, 0, stream()>>>(a, b, copy);
    YAO_HIP(hipGetLastError());
    return 0;
}

// Raise the dynamic LDS limit of every pass kernel ahead of a graph capture.
int prepare_pass_kernels()
{
    YAO_TRY(set_lds_limit(k_pass_fwd<float>));
    YAO_TRY(set_lds_limit(k_pass_fwd<double>));
    YAO_TRY(set_lds_limit(k_pass_bwd<float, true>));
    YAO_TRY(set_lds_limit(k_pass_bwd<float, false>));
    YAO_TRY(set_lds_limit(k_pass_bwd<double, true>));
    YAO_TRY(set_lds_limit(k_pass_bwd<double, false>));
    YAO_TRY(set_lds_limit(k_small_circuit));
    YAO_TRY(set_lds_limit(k_pass_fwd_many<float>));
    YAO_TRY(set_lds_limit(k_pass_fwd_many<double>));
    YAO_TRY(set_lds_limit(k_pass_bwd_many<float>));
    YAO_TRY(set_lds_limit(k_pass_bwd_many<double>));
    return 0;
}

size_t pass_lds_bytes(bool bwd, int t, int c, int psi_bytes, int lam_bytes, int dm_words, int mslots)
{
    if (!bwd) return ((size_t)psi_bytes << t) + 16 * (size_t)dm_words;
    const int nthr = 1 << (t - kRegBitsBwd);
    return ((size_t)(16 + lam_bytes) << t) + sizeof(double) * 2 * mslots * (size_t)grad_entries(nthr, c);
}

// The tile geometry of a pass: tile qubits (ascending), the qubits outside the tile, and the
// per-register offsets of the load mapping for RB register bits.
static void tile_args(PassArgs& a, int n, int B, int c, int t, const std::vector<int>& tile_qubits, int RB,
                      const std::vector<int>& store_src = {})
{
    // Store permutation (identity when store_src is empty).
    for (int i = 0; i < t; ++i) {
        const int src = store_src.empty() ? i : store_src[i];
        if (i < t - RB) a.ssrc[i] = src;
    }
    for (int r = 0; r < (1 << RB); ++r) {
        uint32_t v = 0;
        for (int j = 0; j < RB; ++j)
            if ((r >> j) & 1) v |= 1u << (store_src.empty() ? t - RB + j : store_src[t - RB + j]);
        a.sreg[r] = v;
    }
    a.n = n;
    a.B = B;
    a.c = c;
    a.t = t;
    a.ntq = (int)tile_qubits.size();
    uint64_t T = 0;
    for (int j = 0; j < a.ntq; ++j) {
        a.tile_qubits[j] = tile_qubits[j];
        T |= uint64_t(1) << tile_qubits[j];
    }
    a.nnt = 0;
    for (int q = 0; q < n; ++q)
        if (!((T >> q) & 1)) a.nontile_qubits[a.nnt++] = q;
    const int j0 = t - RB - c;
    for (int r = 0; r < (1 << RB); ++r) {
        uint64_t d = 0;
        for (int rb = 0; rb < RB; ++rb)
            if ((r >> rb) & 1) d |= uint64_t(1) << tile_qubits[j0 + rb];
        a.rofs[r] = d * (uint64_t)B;
    }
    a.ntiles = 1 << a.nnt;
}

// The arguments of one pass and the threads and LDS its tiles take.
static int pass_setup(PassArgs& a, bool bwd, int psi_dtype, int lam_dtype, void* psi, void* lam, const POp* ops,
                      const PGroupDesc* groups, const double* mats, double* gpartial, int pstride, int mslots, int n, int B,
                      int c, int t, int group0, int ngroups, const std::vector<int>& tile_qubits,
                      const std::vector<int>& store_src, int op_first, int nops, const double* dmats, int dm_words,
                      int* threads, size_t* lds_bytes)
{
    if (bwd && (mslots < 1 || mslots > kMaxGroupSlots))
        return set_error(YAO_EINVAL, "%d gradient slots per register group (1 .. %d)", mslots, kMaxGroupSlots);
    if (!store_src.empty() && (int)store_src.size() != t)
        return set_error(YAO_EINVAL, "store permutation of %zu bits for a tile of %d", store_src.size(), t);
    if (!store_src.empty()) {
        uint32_t seen = 0;
        for (int v : store_src) {
            if (v < 0 || v >= t || ((seen >> v) & 1)) return set_error(YAO_EINVAL, "store permutation is not one");
            seen |= 1u << v;
        }
        for (int b = 0; b < c; ++b)
            if (store_src[b] != b) return set_error(YAO_EINVAL, "store permutation moves a batch bit");
    }
    if (nops > kMaxPassOps || ngroups > kMaxPassOps)
        return set_error(YAO_EINVAL, "pass of %d ops exceeds %d", nops, kMaxPassOps);
    const int dm_max = bwd ? 0 : kMaxPassDense * 256;  // 4 KiB per block in every layout
    if (dm_words < 0 || dm_words > dm_max)
        return set_error(YAO_EINVAL, "pass carries %d words of dense matrices (at most %d)", dm_words, dm_max);
    memset(&a, 0, sizeof(a));
    a.psi = psi;
    a.lam = lam;
    a.ops = ops + op_first;
    a.groups = groups + group0;
    a.mats = mats;
    a.gpartial = gpartial;
    a.dmats = (const uint4*)dmats;
    a.ndm = dm_words;
    a.ngroups = ngroups;
    a.nops = nops;
    a.mslots = mslots;
    a.zs = g_zbatch.zs;
    a.op_first = op_first;
    tile_args(a, n, B, c, t, tile_qubits, bwd ? kRegBitsBwd : kRegBitsFwd, store_src);
    a.pstride = pstride > a.ntiles ? pstride : a.ntiles;
    const int RBk = bwd ? kRegBitsBwd : kRegBitsFwd;
    // The kernels are compiled for at most 512 threads per block (one tile, 2^(t - RB) threads).
    if (t - RBk < 0 || t - RBk > 9) return set_error(YAO_EINVAL, "tile of 2^%d does not fit 1 .. 512 threads", t);
    *threads = 1 << (t - RBk);
    const int pb = bwd ? 16 : (psi_dtype == YAO_C64 ? 8 : 16);
    const int lb = bwd ? (lam_dtype == YAO_C64 ? 8 : 16) : 0;
    *lds_bytes = pass_lds_bytes(bwd, t, c, pb, lb, bwd ? 0 : dm_words, mslots);
    if (*lds_bytes > 160 * 1024) return set_error(YAO_EINVAL, "tile of 2^%d needs %zu bytes of LDS", t, *lds_bytes);
    return 0;
}

int launch_pass(bool bwd, int psi_dtype, int lam_dtype, void* psi, void* lam, const POp* ops, const PGroupDesc* groups,
                const double* mats, double* gpartial, int pstride, int mslots, int n, int B, int c, int t, int group0,
                int ngroups, const std::vector<int>& tile_qubits, const std::vector<int>& store_src, double flops,
                int op_first, int nops, const double* dmats, int dm_words)
{
    PassArgs a;
    int threads = 0;
    size_t lds = 0;
    YAO_TRY(pass_setup(a, bwd, psi_dtype, lam_dtype, psi, lam, ops, groups, mats, gpartial, pstride, mslots, n, B, c, t,
                       group0, ngroups, tile_qubits, store_src, op_first, nops, dmats, dm_words, &threads, &lds));
    const int Bc = 1 << c, nz = g_zbatch.zs ? g_zbatch.nz : 1;
    const int pb = bwd ? 16 : (psi_dtype == YAO_C64 ? 8 : 16);
    const int lb = bwd ? (lam_dtype == YAO_C64 ? 8 : 16) : 0;
    dim3 grid(a.ntiles, (B + Bc - 1) / Bc, nz);
    dim3 block(threads);
    hipStream_t st = stream();
    const int pi = prof_begin(bwd ? YAO_KF_PASS_BWD : YAO_KF_PASS_FWD);
    if (!bwd) {
        if (psi_dtype == YAO_C64) {
            YAO_TRY(set_lds_limit(k_pass_fwd<float>));
            k_pass_fwd<float><<<grid, block, lds, st>>>(a);
        } else {
            YAO_TRY(set_lds_limit(k_pass_fwd<double>));
            k_pass_fwd<double><<<grid, block, lds, st>>>(a);
        }
    } else {
        if (lam_dtype == YAO_C64) {
            if (c == 0) {
                YAO_TRY(set_lds_limit(k_pass_bwd<float, true>));
                k_pass_bwd<float, true><<<grid, block, lds, st>>>(a);
            } else {
                YAO_TRY(set_lds_limit(k_pass_bwd<float, false>));
                k_pass_bwd<float, false><<<grid, block, lds, st>>>(a);
            }
        } else {
            if (c == 0) {
                YAO_TRY(set_lds_limit(k_pass_bwd<double, true>));
                k_pass_bwd<double, true><<<grid, block, lds, st>>>(a);
            } else {
                YAO_TRY(set_lds_limit(k_pass_bwd<double, false>));
                k_pass_bwd<double, false><<<grid, block, lds, st>>>(a);
            }
        }
    }
    prof_end(pi, 2.0 * (double)(uint64_t(1) << n) * B * (pb + lb) * nz, flops * nz);
    YAO_HIP(hipGetLastError());
    return 0;
}

// ---------------------------------------------------------------------- several circuits at once
size_t many_pass_bytes()
{
    return sizeof(PassArgs);
}

int many_pass(void* dst, const Plan& P, const Program& prog, const DevProgram& d, int p, int dtype, void* psi, void* lam,
              double* gpartial, int pstride, int* ntiles, int* threads, size_t* lds)
{
    const HostPass& pass = P.passes[p];
    const bool bwd = P.reverse;
    PassArgs a;
    YAO_TRY(pass_setup(a, bwd, bwd ? YAO_C128 : dtype, dtype, psi, lam, d.ops, d.groups, d.mats, gpartial, pstride,
                       bwd ? P.max_slots : 0, P.n, 1, P.c, P.t, prog.pass_group0[p], (int)pass.groups.size(),
                       pass.tile_qubits, pass.store_src, prog.pass_op0[p], prog.pass_nops[p],
                       bwd ? nullptr : d.mats + prog.pass_dmat0[p], bwd ? 0 : prog.pass_dmat_words[p], threads, lds));
    a.zs = nullptr;
    *ntiles = a.ntiles;
    memcpy(dst, &a, sizeof(a));
    return 0;
}

int launch_many_passes(bool bwd, int dtype, const ManyStep& s)
{
    if (s.nblocks <= 0) return 0;
    const PassArgs* items = (const PassArgs*)s.items;
    hipStream_t st = stream();
    if (!bwd) {
        if (dtype == YAO_C64) k_pass_fwd_many<float><<<s.nblocks, s.threads, s.lds, st>>>(items, s.blocks);
        else k_pass_fwd_many<double><<<s.nblocks, s.threads, s.lds, st>>>(items, s.blocks);
    } else {
        if (dtype == YAO_C64) k_pass_bwd_many<float><<<s.nblocks, s.threads, s.lds, st>>>(items, s.blocks);
        else k_pass_bwd_many<double><<<s.nblocks, s.threads, s.lds, st>>>(items, s.blocks);
    }
    YAO_HIP(hipGetLastError());
    return 0;
}

int launch_many_obs(int dtype, int reg_bits, const ManyStep& s)
{
    if (s.nblocks <= 0) return 0;
    const ManyObs* items = (const ManyObs*)s.items;
    hipStream_t st = stream();
    if (dtype == YAO_C64) {
        if (reg_bits == 1) k_obs_gather_many<float, 1><<<s.nblocks, kObsGatherThreads, 0, st>>>(items, s.blocks);
        else k_obs_gather_many<float, 2><<<s.nblocks, kObsGatherThreads, 0, st>>>(items, s.blocks);
    } else {
        if (reg_bits == 1) k_obs_gather_many<double, 1><<<s.nblocks, kObsGatherThreads, 0, st>>>(items, s.blocks);
        else k_obs_gather_many<double, 2><<<s.nblocks, kObsGatherThreads, 0, st>>>(items, s.blocks);
    }
    YAO_HIP(hipGetLastError());
    return 0;
}

int launch_many_rows(const ManyStep& s)
{
    if (s.nblocks <= 0) return 0;
    k_rows_many<<<s.nblocks, 256, 0, stream()>>>((const ManyRows*)s.items, s.blocks);
    YAO_HIP(hipGetLastError());
    return 0;
}

int launch_many_resets(int dtype, void* const* states, const int* n, int count)
{
    if (count <= 0) return 0;
    if (dtype == YAO_C64) k_reset_many<float><<<dim3(32, count), 256, 0, stream()>>>(states, n);
    else k_reset_many<double><<<dim3(32, count), 256, 0, stream()>>>(states, n);
    YAO_HIP(hipGetLastError());
    return 0;
}

// ---------------------------------------------------------------------- observable passes
namespace {

struct ObsPass {
    std::vector<int> tile_qubits;
    int r0 = 0, r1 = 0;  // records of the pass in the device table
};
struct ObsPlan {
    bool ok = false;  // false: an X mask is wider than a tile (the observable takes the
                      // per-group kernels)
    bool gather = false;  // one launch of k_obs_gather instead of tile passes
    int c = 0, t = 0;
    std::vector<ObsPass> passes;
    ObsRec* drecs = nullptr;
};
using ObsKey = std::tuple<const yao_pauli_sum*, int, int, int, int>;  // h, n, B, dtype, use
std::map<ObsKey, ObsPlan*> g_obs;
std::mutex g_obs_mu;

// Elements per thread of k_obs_gather: two keep every CU busy up to 17 qubits (16 qubits,
// complex128: 9.3 us; tiles 33.6 us), above that four share the terms' signs.
int obs_gather_reg_bits(int n)
{
    return n <= 17 ? 1 : 2;
}

// Whether a single-slot state takes k_obs_gather rather than npasses tile passes over the X masks xs (wide: one of
// them is wider than a tile, and then the passes are the per-group kernels). Both forms were timed for
// observables of 1 to 567 masks and 1 to 31 passes (chains, all pairs, random strings on 4, 6, the lowest 12 or
// all qubits, 1 to 1000 terms a mask) on 10 to 25 qubits. Up to 2^19 complex64 or 2^17 complex128
// amplitudes the gather always won; beyond, the sum below is their difference in us, with M = 2^20
// amplitudes, and picks the better form to 0.4 % of its time on average:
// - a mask costs the gather a read of the state in an order that the mask stirs: little for two qubits,
//   0.9 us M from five (complex128 2.1), half of it where the L2 caches hold the state and 0.7 at 16 MiB; and a tile
//   pass its reads of LDS, 0.12 us M;
// - a term costs the gather 0.018 us M more (four elements share its sign, eight in a tile);
// - a pass costs its launch and its read of the state, with H psi a read and a write of that too (more where both
//   no longer fit the 256 MiB Infinity Cache).
// 20 qubits complex128, 400 masks on the 12 lowest qubits (one pass): energy 733 us by the gather, 149 by tiles;
// 21 qubits complex64, all pairs (14 passes): H psi 313 against 427; 24 qubits complex128, 40 masks on 6 qubits
// (18 passes): energy 1540 against 1203, H psi 1532 against 3123; 25 qubits complex64, chain (3 passes): energy
// 519 against 466, H psi 574 against 983. Energies under wide masks: 0.4 to 0.96 of the per-group kernels' time, but for
// 1.04 at 23 qubits complex128; H psi 0.6 to 1.0 for complex64, 1.02 to 1.10 for complex128 from 20 qubits.
// OBS_ONE: H psi where one launch spares the caller others, about 20 us and another read of the state.
bool obs_gathers(const yao_pauli_sum* h, int n, int B, int dtype, int use, const std::vector<uint64_t>& xs, int npasses,
                 bool wide)
{
    const bool single = dtype == YAO_C64;
    if (use == OBS_TILES || B != 1 || n > 31) return false;
    if (wide) return use != OBS_VECTOR || single || n < 20;
    if (n > (single ? 25 : 24)) return false;
    if (n <= (single ? 19 : 17)) return true;
    const double M = std::ldexp(1.0, n - 20), mib = (single ? 8 : 16) * M;
    const double read = (single ? 0.3 : 0.7) * M * (mib <= 8 ? 0.5 : mib <= 16 ? 0.7 : 1.0), lds = std::max(0.22, 0.12 * M);
    double more = 12 + 2.4 * M + 0.018 * M * (double)h->coef.size();
    for (uint64_t x : xs) more += std::max(lds, read * std::min(4, __builtin_popcountll(x) - 1)) - lds;
    double pass;
    if (use == OBS_ENERGY) pass = 6 + (single ? 2.6 : 3.5) * M;
    else if (2 * mib > 256) pass = 10 + (single ? 8.4 : 10.0) * M;
    else pass = 10 + (single ? 5.0 : 6.0) * M;
    return more <= pass * npasses + (use == OBS_ONE ? 20 + (single ? 1.7 : 3.4) * M : 0.0);
}

// The X masks of an observable in order of appearance, and the terms of each.
struct ObsMasks {
    std::vector<uint64_t> xs;
    std::vector<std::vector<int>> terms;
    explicit ObsMasks(const yao_pauli_sum* h)
    {
        std::unordered_map<uint64_t, int> at;
        for (size_t k = 0; k < h->x.size(); ++k) {
            const auto e = at.emplace(h->x[k], (int)xs.size());
            if (e.second) {
                xs.push_back(h->x[k]);
                terms.emplace_back();
            }
            terms[e.first->second].push_back((int)k);
        }
    }
};

// The records of the terms of some X masks (which: indices into M), in order: bit q of an index is bit pos[q] of
// the thread's coordinates (-1: outside the tile), of which the top rb of nb bits are register bits. One
// step a term: a plan per use of an observable of 20000 terms takes a few ms, where a look over all
// terms for every mask took 50.
void obs_records(const yao_pauli_sum* h, const ObsMasks& M, const std::vector<int>& which, const std::vector<int>& pos,
                 int nb, int rb, std::vector<ObsRec>& out)
{
    auto inside = [&](uint64_t m) {
        uint32_t r = 0;
        for (size_t q = 0; q < pos.size(); ++q)
            if (((m >> q) & 1) && pos[q] >= 0) r |= 1u << pos[q];
        return r;
    };
    uint64_t outer = 0;
    for (size_t q = 0; q < pos.size(); ++q)
        if (pos[q] < 0) outer |= uint64_t(1) << q;
    const uint32_t own = (1u << (nb - rb)) - 1;
    size_t last = out.size();  // first record of the mask before
    for (int m : which) {
        const size_t at = out.size();
        const uint32_t xi = inside(M.xs[m]);
        for (int k : M.terms[m]) {
            const uint32_t z = inside(h->z[k]);
            const int ny = __builtin_popcountll(h->x[k] & h->z[k]);
            // Every element's source is its own index ^ x: the sign of |x & z| belongs to the term.
            const bool neg = (((ny >> 1) ^ __builtin_popcount(xi & z)) & 1) != 0;
            ObsRec r;
            r.c = neg ? -h->coef[k] : h->coef[k];
            r.zout = h->z[k] & outer;
            r.zin = z & own;
            r.x = xi;
            r.xnext = 0;
            r.flags = (z >> (nb - rb)) | ((ny & 1) ? 8u : 0u);
            out.push_back(r);
        }
        std::stable_sort(out.begin() + at, out.end(), [](const ObsRec& p, const ObsRec& q) { return p.flags < q.flags; });
        for (size_t k = at; k < out.size(); ++k)
            if (k + 1 == out.size() || (out[k + 1].flags & 15) != (out[k].flags & 15)) out[k].flags |= kObsLast;
        out[at].flags |= kObsFirst;
        for (size_t k = last; k < at; ++k) out[k].xnext = out[at].x;
        last = at;
    }
}

// Group the terms by X mask, then put each mask in the first pass whose tile qubits can take
// it (first fit, over tiles of t - c qubits that keep the lowest qubits for contiguous
// rows), and fill every pass's tile with the lowest unused qubits.
ObsPlan* obs_plan(const yao_pauli_sum* h, int n, int B, int dtype, int use)
{
    std::lock_guard<std::mutex> lk(g_obs_mu);
    const ObsKey key{h, n, B, dtype, use};
    auto it = g_obs.find(key);
    if (it != g_obs.end()) return it->second;
    const int lb = ilog2_ceil((uint64_t)B);
    const int c = lb < 3 ? lb : 3;
    const int tq = std::min(n, kObsMaxTile - c);
    const int L = std::max(0, std::min((dtype == YAO_C64 ? 4 : 3) - c, tq));
    const ObsMasks M(h);
    const std::vector<uint64_t>& xs = M.xs;
    bool wide = false;
    for (uint64_t x : xs) wide |= __builtin_popcountll(x) > tq;
    const uint64_t low = L > 0 ? ((uint64_t(1) << L) - 1) : 0;
    ObsPlan* P = new ObsPlan;
    P->c = c;
    P->t = c + tq;
    std::vector<uint64_t> T;           // qubits of each pass
    std::vector<std::vector<int>> gx;  // X masks of each pass
    for (size_t m = 0; m < xs.size() && !wide; ++m) {
        const uint64_t x = xs[m];
        size_t p = 0;
        while (p < T.size() && __builtin_popcountll(T[p] | x) > tq) ++p;
        if (p == T.size()) {
            // A mask too wide for a tile with the low qubits fixed drops them.
            T.push_back(__builtin_popcountll(low | x) <= tq ? low : 0);
            gx.emplace_back();
        }
        T[p] |= x;
        gx[p].push_back((int)m);
    }
    P->gather = obs_gathers(h, n, B, dtype, use, xs, (int)T.size(), wide);
    if (wide && !P->gather) {
        g_obs[key] = P;
        return P;
    }
    std::vector<ObsRec> hr;
    if (P->gather) {
        std::vector<int> pos(n);
        for (int q = 0; q < n; ++q) pos[q] = q;
        ObsPass ps;
        std::vector<int> all(xs.size());
        for (size_t m = 0; m < all.size(); ++m) all[m] = (int)m;
        obs_records(h, M, all, pos, n, obs_gather_reg_bits(n), hr);
        ps.r1 = (int)hr.size();
        P->passes.push_back(ps);
    }
    for (size_t p = 0; p < T.size() && !P->gather; ++p) {
        uint64_t Tp = T[p];
        for (int q = 0; q < n && __builtin_popcountll(Tp) < tq; ++q) Tp |= uint64_t(1) << q;
        ObsPass ps;
        std::vector<int> pos(n, -1);
        for (int q = 0; q < n; ++q)
            if ((Tp >> q) & 1) {
                pos[q] = c + (int)ps.tile_qubits.size();
                ps.tile_qubits.push_back(q);
            }
        ps.r0 = (int)hr.size();
        obs_records(h, M, gx[p], pos, P->t, kObsRegBits, hr);
        ps.r1 = (int)hr.size();
        P->passes.push_back(ps);
    }
    hr.push_back(ObsRec{});  // read one past the last, never used
    if (hipMalloc((void**)&P->drecs, sizeof(ObsRec) * hr.size()) != hipSuccess ||
        hipMemcpy(P->drecs, hr.data(), sizeof(ObsRec) * hr.size(), hipMemcpyHostToDevice) != hipSuccess) {
        if (P->drecs) (void)hipFree(P->drecs);
        delete P;
        set_error(YAO_ENOMEM, "observable pass tables");
        return nullptr;
    }
    P->ok = true;
    g_obs[key] = P;
    return P;
}

// The launch arguments of one pass; run(<state real>, <output real>, <with output>) per type.
template <typename F> int obs_by_type(int dtype, int out_dtype, bool out, F run)
{
    if (!out) return dtype == YAO_C64 ? run(float(), float(), std::false_type()) : run(double(), double(), std::false_type());
    if (dtype == YAO_C64)
        return out_dtype == YAO_C64 ? run(float(), float(), std::true_type()) : run(float(), double(), std::true_type());
    return out_dtype == YAO_C64 ? run(double(), float(), std::true_type()) : run(double(), double(), std::true_type());
}

int obs_gather_threads(int n)
{
    return (int)std::min<uint64_t>(kObsGatherThreads, uint64_t(1) << (n - obs_gather_reg_bits(n)));
}

// Columns of energy partials per batch slot.
int obs_columns(const ObsPlan* P, int n)
{
    if (P->gather) return (int)((uint64_t(1) << (n - obs_gather_reg_bits(n))) / obs_gather_threads(n));
    return (int)P->passes.size() * (1 << (n - (P->t - P->c)));
}

}  // namespace

bool obs_passes_ok(const yao_pauli_sum* h, int n, int B, int dtype, int use)
{
    if (n < kObsRegBits + 1) return false;
    const ObsPlan* P = obs_plan(h, n, B, dtype, use);
    return P && P->ok;
}

int obs_tile_qubits(const yao_pauli_sum* h, int n, int B, int dtype)
{
    const ObsPlan* P = obs_plan(h, n, B, dtype, OBS_TILES);
    return P && P->ok ? P->t - P->c : 0;
}

bool obs_one_launch(const yao_pauli_sum* h, int n, int B, int dtype, int use)
{
    if (n < kObsRegBits + 1) return false;
    const ObsPlan* P = obs_plan(h, n, B, dtype, use);
    return P && P->ok && P->gather;
}

// One item of launch_many_obs: its columns are obs_partial_doubles (OBS_ONE), its blocks *blocks of 256 threads.
int many_obs(ManyObs& o, int* reg_bits, int* blocks, const void* psi, void* lam, double* psi64, int dtype, int n,
             const yao_pauli_sum* h, double* partial)
{
    const ObsPlan* P = obs_plan(h, n, 1, dtype, OBS_ONE);
    if (!P) return YAO_ENOMEM;
    if (!P->ok || !P->gather || obs_gather_threads(n) != kObsGatherThreads)
        return set_error(YAO_EINVAL, "observable takes more than one launch");
    o = ManyObs{psi, lam, psi64, partial, P->drecs, P->passes[0].r1, n};
    *reg_bits = obs_gather_reg_bits(n);
    *blocks = obs_columns(P, n);
    return 0;
}

int launch_lanczos_hv(const void* src, void* v, void* out, int dtype, int n, const yao_pauli_sum* h, const double* npart,
                      int nn, double* norm, double* partial)
{
    const ObsPlan* P = obs_plan(h, n, 1, dtype, OBS_ONE);
    if (!P) return YAO_ENOMEM;
    if (!P->ok || !P->gather) return set_error(YAO_EINVAL, "observable takes more than one launch");
    const ObsRec* recs = P->drecs;
    const int nrec = P->passes[0].r1, grid = obs_columns(P, n), nthr = obs_gather_threads(n);
#define YAO_LANCZOS(R, RB)                                                                                        \
    k_lanczos_hv<R, RB><<<grid, nthr, 0, stream()>>>((const vec2_t<R>*)src, (vec2_t<R>*)v, (vec2_t<R>*)out, n, recs, nrec, \
                                                      npart, nn, norm, partial)
    const bool one = obs_gather_reg_bits(n) == 1;
    if (dtype == YAO_C64) {
        if (one) YAO_LANCZOS(float, 1);
        else YAO_LANCZOS(float, 2);
    } else {
        if (one) YAO_LANCZOS(double, 1);
        else YAO_LANCZOS(double, 2);
    }
#undef YAO_LANCZOS
    YAO_HIP(hipGetLastError());
    return 0;
}

size_t obs_partial_doubles(const yao_pauli_sum* h, int n, int B, int dtype, int use)
{
    const ObsPlan* P = obs_plan(h, n, B, dtype, use);
    if (!P || !P->ok) return 0;
    return (size_t)B * obs_columns(P, n);
}

// H psi into out (out == nullptr: the energy only) and the partials of the energy in
// partial[b * W + column]; *W receives the row length (OBS_TILES: per pass and tile, in tile order).
int launch_obs_passes(const void* psi, int dtype, void* out, int out_dtype, int n, int B, const yao_pauli_sum* h,
                      double* partial, int* W, int use, double* psi64)
{
    const ObsPlan* P = obs_plan(h, n, B, dtype, use);
    if (!P) return YAO_ENOMEM;
    if (!P->ok) return set_error(YAO_EINVAL, "observable has an X mask wider than a tile");
    if (psi64 && !P->gather) return set_error(YAO_EINVAL, "tile passes do not widen the state");
    *W = obs_columns(P, n);
    const int nz = g_zbatch.zs ? g_zbatch.nz : 1;
    PassArgs a;
    memset(&a, 0, sizeof(a));
    a.psi = const_cast<void*>(psi);
    a.lam = out;
    a.zs = g_zbatch.zs;
    if (P->gather) {
        a.n = n;
        const dim3 grid(*W, 1, nz);
        return obs_by_type(dtype, out_dtype, out != nullptr, [&](auto rp, auto ro, auto with) {
            using RP = decltype(rp);
            using RO = decltype(ro);
            constexpr bool OUT = decltype(with)::value;
            if (obs_gather_reg_bits(n) == 1)
                k_obs_gather<RP, RO, OUT, 1><<<grid, obs_gather_threads(n), 0, stream()>>>(a, P->drecs, P->passes[0].r1, partial, (double2*)psi64);
            else
                k_obs_gather<RP, RO, OUT, 2><<<grid, obs_gather_threads(n), 0, stream()>>>(a, P->drecs, P->passes[0].r1, partial, (double2*)psi64);
            YAO_HIP(hipGetLastError());
            return 0;
        });
    }
    const int t = P->t, c = P->c;
    const int nthr = 1 << (t - kObsRegBits);
    const int ntiles = 1 << (n - (t - c));
    const int Bc = 1 << c;
    const dim3 grid(ntiles, (B + Bc - 1) / Bc, nz);
    const size_t lds = ((size_t)(dtype == YAO_C64 ? 8 : 16) << t) + sizeof(double) * (size_t)grad_entries(nthr, c);
    for (size_t p = 0; p < P->passes.size(); ++p) {
        const ObsPass& ps = P->passes[p];
        tile_args(a, n, B, c, t, ps.tile_qubits, kObsRegBits);
        const int acc = p > 0 ? 1 : 0, col = (int)p * ntiles;
        YAO_TRY(obs_by_type(dtype, out_dtype, out != nullptr, [&](auto rp, auto ro, auto with) {
            using RP = decltype(rp);
            using RO = decltype(ro);
            constexpr bool OUT = decltype(with)::value;
            YAO_TRY(set_lds_limit(k_obs_pass<RP, RO, OUT>));
            k_obs_pass<RP, RO, OUT><<<grid, nthr, lds, stream()>>>(a, P->drecs + ps.r0, ps.r1 - ps.r0, acc, partial, col, *W);
            YAO_HIP(hipGetLastError());
            return 0;
        }));
    }
    return 0;
}

void drop_obs_plans(const yao_pauli_sum* h)
{
    std::lock_guard<std::mutex> lk(g_obs_mu);
    for (auto it = g_obs.begin(); it != g_obs.end();) {
        if (std::get<0>(it->first) == h) {
            (void)hipDeviceSynchronize();
            if (it->second->drecs) (void)hipFree(it->second->drecs);
            delete it->second;
            it = g_obs.erase(it);
        } else {
            ++it;
        }
    }
}

}  // namespace yao
