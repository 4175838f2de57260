// Run-time compiled pass kernels (hipRTC). The generic pass kernels read every op record at run
// time and dispatch on its variant: per op, scalar loads, a compare tree, loop control and, at
// the merge of the variants, register copies. With one wave per SIMD (a 20-qubit state gives
// each CU one 2^12 tile) that scalar work is not hidden behind another wave's vector work. A
// device-bound program's structure (which ops, on which register bits, under which controls)
// is fixed; only its matrices change with the parameters, and they stay in the op records that
// k_bind rewrites. So each pass of such a program can be emitted as straight-line code: the
// tile mapping and the register-group layouts become constants, a SWAP on register bits whose
// controls are register bits is a renaming of registers at compile time (no instructions),
// and the matrix entries are read from the records at constant offsets.
//
// Supported: passes whose groups are all register groups (no
// LDS-applied k = 2, 3 ops and no dense blocks); the LDS of a compiled pass is a static
// allocation of the sizes the pass needs. Any other pass of the program runs the generic
// kernel. A compile failure switches the program back to the generic kernels for good.
#include <hip/hiprtc.h>

#include <algorithm>
#include <cstdio>
#include <atomic>
#include <cstddef>
#include <mutex>
#include <sstream>
#include <string>
#include <thread>
#include <vector>

#include "fused.h"

namespace yao {

namespace {

std::string I(long long v)
{
    return std::to_string(v);
}
std::string U(unsigned long long v)
{
    return std::to_string(v) + "ull";
}

// Bank swizzle of the LDS tile, linear over GF(2): row e lies at e with its low 5 bits (the banks of
// 8-byte rows; the low 4 are those of 16-byte rows) XORed with a column per high bit. The columns were
// searched so that the tile bits outside a register group, any 2 to 4 bits taken out of 12 (780 of
// 781 choices), hold 5 whose images are independent: lane_order puts those on the lowest lanes, so
// that a wave's accesses of the tile meet every bank once. 25 qubits, depth 20, complex64, SQ counters of 126
// passes: 9.9e9 LDS cycles with the generic kernels' swizzle and the tile bits in order, 4.4e9 of them
// conflicts; 6.9e9 and 2.8e9 now (with the matrices' reads and the loads' and stores' own order).
uint32_t swz_host(uint32_t e)
{
    static const uint32_t col[8] = {26, 7, 22, 21, 3, 28, 13, 19};
    uint32_t v = e;
    for (int b = 5; b < 13; ++b)
        if ((e >> b) & 1) v ^= col[b - 5];
    return v;
}

int gf2_rank(std::vector<uint32_t> v)
{
    int r = 0;
    for (size_t i = 0; i < v.size(); ++i) {
        if (!v[i]) continue;
        ++r;
        const uint32_t low = v[i] & (0u - v[i]);
        for (size_t j = i + 1; j < v.size(); ++j)
            if (v[j] & low) v[j] ^= v[i];
    }
    return r;
}

// The tile bits outside the mask regs in the order of the thread bits that address them: 4 whose
// images are independent in the low 4 bits, then one that adds the fifth bank bit, then the rest (the
// choice of most independent images where no such 5 exist).
// The c batch bits, the tile's lowest and their own images, stay on the lowest lanes.
std::vector<int> lane_order(int t, int c, uint32_t regs)
{
    std::vector<int> bits;
    for (int b = 0; b < t; ++b)
        if (!((regs >> b) & 1)) bits.push_back(b);
    const int m = (int)bits.size();
    if (m < 4) return bits;
    std::vector<int> best = bits;
    int best_rank = -1;
    for (uint32_t pick = 0; pick < (1u << m) && best_rank < 9; ++pick) {
        if (__builtin_popcount(pick) != 4 || (pick & ((1u << c) - 1)) != (1u << c) - 1) continue;
        std::vector<int> order;
        std::vector<uint32_t> low4, low5;
        for (int i = 0; i < m; ++i)
            if ((pick >> i) & 1) {
                order.push_back(bits[i]);
                low4.push_back(swz_host(1u << bits[i]) & 15u);
                low5.push_back(swz_host(1u << bits[i]) & 31u);
            }
        const int r4 = gf2_rank(low4);
        int fifth = -1, r5 = gf2_rank(low5);
        for (int i = 0; i < m && fifth < 0; ++i) {
            if ((pick >> i) & 1) continue;
            std::vector<uint32_t> v = low5;
            v.push_back(swz_host(1u << bits[i]) & 31u);
            if (gf2_rank(v) > r5) fifth = bits[i];
        }
        if (fifth >= 0) {
            order.push_back(fifth);
            ++r5;
        }
        if (r4 + r5 <= best_rank) continue;
        best_rank = r4 + r5;
        for (int b : bits)
            if (std::find(order.begin(), order.end(), b) == order.end()) order.push_back(b);
        best = order;
    }
    return best;
}

// Code that declares `name` as the LDS position of the thread's tile bits: thread bit k on tile bit at[k].
std::string thread_position(const std::string& name, const std::vector<int>& at)
{
    std::string o = "unsigned " + name + " = 0;";
    for (size_t k = 0; k < at.size(); ++k)
        o += " " + name + " ^= (0u - ((th >> " + std::to_string(k) + ") & 1u)) & " +
             std::to_string(swz_host(1u << at[k])) + "u;";
    return o + "\n";
}

// Pointers in the generated code carry their address space: global memory for states and
// partials (global instead of flat loads) and constant for the op records (scalar loads).
const char* kPrelude = R"YAO(
typedef unsigned long long u64;
#define GLB __attribute__((address_space(1)))
#define CST __attribute__((address_space(4)))
#define LDS __attribute__((address_space(3)))
typedef float v4f __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float2 flip(float2 a, unsigned s)
{
    return make_float2(__builtin_bit_cast(float, __builtin_bit_cast(unsigned, a.x) ^ s),
                       __builtin_bit_cast(float, __builtin_bit_cast(unsigned, a.y) ^ s));
}
__device__ __forceinline__ double2 flip(double2 a, unsigned s)
{
    return make_double2(__builtin_bit_cast(double, __builtin_bit_cast(u64, a.x) ^ ((u64)s << 32)),
                        __builtin_bit_cast(double, __builtin_bit_cast(u64, a.y) ^ ((u64)s << 32)));
}
)YAO";

// How an op changes a pair (p, q), as expressions in its matrix entries u[0..7] (re[4], im[4]): the
// structure class of its matrix says which entries are zero; an empty expression leaves the
// amplitude alone. neg: q changes sign. fixed: the entries do not depend on parameters, so d0 = 1 and
// d1 = -1 of a diagonal can be relied on (Z, S, T and phase gates under any controls).
struct PairUpdate {
    std::string p, q;
    bool neg = false;
    std::vector<int> entries;  // entries of u that p and q read
};
PairUpdate pair_update(int type, const std::string& MK, const double* u, bool fixed)
{
    PairUpdate x;
    switch (type) {
    case OT_SWAP:
        x.p = "q";
        x.q = "p";
        break;
    case OT_DIAG:
        if (!(fixed && u[0] == 1 && u[4] == 0)) {
            x.p = MK + "(u[0] * p.x - u[4] * p.y, u[0] * p.y + u[4] * p.x)";
            x.entries = {0, 4};
        }
        if (fixed && u[3] == -1 && u[7] == 0) {
            x.neg = true;
        } else {
            x.q = MK + "(u[3] * q.x - u[7] * q.y, u[3] * q.y + u[7] * q.x)";
            x.entries.insert(x.entries.end(), {3, 7});
        }
        break;
    case OT_REAL:
        x.p = MK + "(u[0] * p.x + u[1] * q.x, u[0] * p.y + u[1] * q.y)";
        x.q = MK + "(u[2] * p.x + u[3] * q.x, u[2] * p.y + u[3] * q.y)";
        x.entries = {0, 1, 2, 3};
        break;
    case OT_RX:  // (c a + i s b, i s a + c b), c = u[0], s = u[5]
        x.p = MK + "(u[0] * p.x - u[5] * q.y, u[0] * p.y + u[5] * q.x)";
        x.q = MK + "(u[0] * q.x - u[5] * p.y, u[0] * q.y + u[5] * p.x)";
        x.entries = {0, 5};
        break;
    default:
        x.p = MK + "(u[0] * p.x - u[4] * p.y + u[1] * q.x - u[5] * q.y, u[0] * p.y + u[4] * p.x + u[1] * q.y + u[5] * q.x)";
        x.q = MK + "(u[2] * p.x - u[6] * p.y + u[3] * q.x - u[7] * q.y, u[2] * p.y + u[6] * p.x + u[3] * q.y + u[7] * q.x)";
        x.entries = {0, 1, 2, 3, 4, 5, 6, 7};
        break;
    }
    return x;
}

// The statement that applies x to registers A and B of type V, under the lane or tile predicate pc
// when cond (sm: the sign bit where pc holds).
std::string pair_code(const PairUpdate& x, const std::string& V, const std::string& A, const std::string& B, bool cond)
{
    std::string o = "      { const " + V + " p = " + A + ", q = " + B + "; ";
    if (!x.p.empty()) o += A + " = " + (cond ? "pc ? " + x.p + " : p; " : x.p + "; ");
    if (x.neg) o += cond ? B + " = flip(q, sm); " : B + ".x = -q.x; " + B + ".y = -q.y; ";
    else if (!x.q.empty()) o += B + " = " + (cond ? "pc ? " + x.q + " : q; " : x.q + "; ");
    return o + "}\n";
}

// The matrix entries of a record as doubles, in program order whatever its precision, and whether
// parameters write them.
void record_entries(const POp& op, bool floats, double* u)
{
    for (int e = 0; e < 8; ++e) u[e] = floats ? (double)((const float*)op.u)[e] : op.u[e];
}
std::vector<char> bound_ops(const Program& prog)
{
    std::vector<char> b(prog.ops.size(), 0);
    for (const BindRec& r : prog.binds) b[r.op] = 1;
    return b;
}

// Code that declares base (the index bits outside the tile), toff (the element of the thread's register
// 0) and, for batches, b0 and bl (the tile's first slot and the thread's place among them), and the
// element offset of each register. Thread bits: the c batch bits, then tile qubits; register bits: the
// next tile qubits. Slots past the batch read its last slot.
std::string tile_code(const Plan& P, const HostPass& pass, int n, std::vector<uint64_t>& rofs)
{
    const int RB = P.reg_bits, N = 1 << RB, t = P.t, c = P.c;
    uint64_t T = 0;
    for (int q : pass.tile_qubits) T |= uint64_t(1) << q;
    std::ostringstream o;
    o << "  const u64 tid = blockIdx.x;\n  u64 base = 0;\n";
    int j = 0;
    for (int q = 0; q < n; ++q)
        if (!((T >> q) & 1)) o << "  base |= ((tid >> " << j++ << ") & 1ull) << " << q << ";\n";
    o << "  u64 toff = base;\n";
    for (int k = 0; k < t - RB - c; ++k)
        o << "  toff |= (u64)((th >> " << c + k << ") & 1u) << " << pass.tile_qubits[k] << ";\n";
    if (P.B > 1)
        o << "  const unsigned b0 = blockIdx.y << " << c << ", bl = th & " << (1 << c) - 1 << "u;\n"
          << "  toff = toff * " << P.B << "ull + (b0 + bl < " << P.B << "u ? b0 + bl : " << P.B - 1 << "u);\n";
    rofs.assign(N, 0);
    for (int r = 0; r < N; ++r)
        for (int b = 0; b < RB; ++b)
            if ((r >> b) & 1) rofs[r] += (uint64_t(1) << pass.tile_qubits[t - RB - c + b]) * (uint64_t)P.B;
    return o.str();
}

// Code of one forward pass, or an empty string when the pass is not supported.
//
// Vector issue bounds complex64 passes of a few gates a qubit (8 instructions an amplitude for a
// merged gate; the 25-qubit depth-20 ansatz needs 3.4 ms of them). An uncontrolled dense gate of a
// compiled plan runs on the matrix cores instead, as the real 4 x 4 product of v_mfma_f32_4x4x1: a
// lane's own pair (re p, im p, re q, im q) is its column of B and D, so no amplitude moves, and 4
// instructions of 8 cycles replace 16 of 4. (Rx-like and diagonal gates cost both the same. Two gates
// as one complex 4 x 4 product cost the same as two real ones.) 25 qubits, depth 20: 4.52 to 4.30 ms, the
// 20-qubit sweep 237 to 219 us: the passes issue a third of the vector instructions (5.1e9 for 15.2e9 over
// 126 passes) beside 25e9 cycles of the matrix cores, 0.32 and 0.39 of a 206 us pass on every SIMD.
std::string gen_forward_pass(const Plan& P, const Program& prog, int p, int n, int dtype, const std::string& name,
                             int* nthr_out, size_t* lds_out)
{
    const HostPass& pass = P.passes[p];
    const int RB = P.reg_bits, N = 1 << RB, t = P.t;
    if (pass.standalone >= 0 || prog.pass_dmat_words[p] != 0) return "";
    if (t - RB < P.c || t - RB > 10 || (int)pass.tile_qubits.size() != t - P.c) return "";
    const int g0 = prog.pass_group0[p], ng = (int)pass.groups.size();
    for (int g = 0; g < ng; ++g)
        if (prog.groups[g0 + g].lds) return "";
    const bool c64 = dtype == YAO_C64;
    const size_t lds = (size_t)(c64 ? 8 : 16) << t;
    if (lds > 160 * 1024) return "";
    const int nthr = 1 << (t - RB);
    const std::string V = c64 ? "float2" : "double2", R = c64 ? "float" : "double";
    const std::string MK = c64 ? "make_float2" : "make_double2";
    const std::vector<char> bound = bound_ops(prog);
    std::ostringstream o;
    // With at most 256 registers a lane the compiler gives matrix instructions vector registers (with
    // accumulation registers every result is moved before its use).
    const std::string waves = c64 && P.compiled ? "__attribute__((amdgpu_waves_per_eu(" + I(RB > 3 ? 3 : 4) + "))) " : "";
    o << "extern \"C\" __global__ void __launch_bounds__(" << nthr << ") " << waves << name
      << "(void* psi_, const char* ops_, const char* zs_, int op_first) {\n";
    // LDS sized at compile time (static allocations may exceed the 64 KiB of a dynamic one):
    // the tile, and the pass's one-qubit matrices (8 entries per record), copied in with the
    // tile so that the ops read them from LDS instead of waiting on a scalar load each.
    const int nrec = prog.pass_nops[p];
    const int UM = c64 && P.compiled ? 16 : 8;  // reals of a record's matrix in LDS
    o << "  __shared__ __align__(16) " << V << " lp[" << (1 << t) << "];\n";
    o << "  __shared__ __align__(16) " << R << " um[" << std::max(1, nrec) * UM << "];\n";
    o << "  const unsigned th = threadIdx.x;\n";
    o << "  GLB " << V << "* gp = (GLB " << V << "*)psi_;\n  const CST char* ops = (const CST char*)ops_;\n";
    o << "  if (zs_) { const CST u64* z = (const CST u64*)(zs_ + 32 * blockIdx.z); gp = (GLB " << V
      << "*)z[0]; ops = (const CST char*)z[2] + (u64)op_first * " << sizeof(POp) << "; }\n";
    std::vector<uint64_t> rofs;
    o << tile_code(P, pass, n, rofs);
    o << "  {\n";
    for (int r = 0; r < N; ++r) o << "    const " << V << " v" << r << " = gp[toff + " << U(rofs[r]) << "];\n";
    {
        const int W = c64 ? UM : 16;  // dwords of a record's matrix
        o << "    { const CST unsigned* src = (const CST unsigned*)ops; unsigned* dst = (unsigned*)um;\n"
          << "      for (unsigned i = th; i < " << nrec * W << "u; i += " << nthr << "u) dst[i] = src[(i / " << W << "u) * "
          << sizeof(POp) / 4 << "u + " << offsetof(POp, u) / 4 << "u + i % " << W << "u]; }\n";
    }
    std::vector<int> thread_bits(t - RB);
    for (int k = 0; k < t - RB; ++k) thread_bits[k] = k;
    // Positions are kept in bytes, one XOR an access.
    const int es = c64 ? 8 : 16;
    auto at = [&](const std::string& pos, uint32_t e) {
        return "*(LDS " + V + "*)((LDS char*)lp + (" + pos + " ^ " + I((long long)swz_host(e) * es) + "u))";
    };
    o << "    " << thread_position("lpos", thread_bits) << "    lpos *= " << es << "u;\n";
    for (int r = 0; r < N; ++r) o << "    " << at("lpos", (uint32_t)r * nthr) << " = v" << r << ";\n";
    o << "  }\n  __syncthreads();\n";
    // Register groups (records are addressed relative to the pass's first record).
    for (int g = 0; g < ng; ++g) {
        const PGroupDesc& G = prog.groups[g0 + g];
        uint32_t rmask = 0;
        for (int j = 0; j < RB; ++j) rmask |= 1u << G.rpos[j];
        std::vector<uint32_t> er(N);
        for (int r = 0; r < N; ++r) {
            uint32_t e = 0;
            for (int j = 0; j < RB; ++j)
                if ((r >> j) & 1) e |= 1u << G.rpos[j];
            er[r] = e;
        }
        const std::vector<int> lanes = lane_order(t, P.c, rmask);
        o << "  {\n    unsigned ethr = 0;\n";
        for (size_t k = 0; k < lanes.size(); ++k) o << "    ethr |= ((th >> " << k << ") & 1u) << " << lanes[k] << ";\n";
        o << "    " << thread_position("sw", lanes) << "    sw *= " << es << "u;\n";
        std::vector<int> perm(N);
        for (int r = 0; r < N; ++r) {
            perm[r] = r;
            o << "    " << V << " x" << r << " = " << at("sw", er[r]) << ";\n";
        }
        for (int i = 0; i < G.nops; ++i) {
            const int oi = G.op0 + i;
            const POp& op = prog.ops[prog.pass_op0[p] + oi];
            const int J = op.rpos;
            const int cls = op.var / RB;
            const uint32_t tm = op.cmask & ~rmask, rm = op.cmask & rmask;
            if (c64 && takes_real_form(P, op)) {
                o << "    {\n      const v4f w = *(const v4f*)(um + " << oi * UM << " + (th & 3u) * 4u);\n";
                std::vector<std::pair<int, int>> pr;
                for (int a = 0; a < N; ++a)
                    if (!((a >> J) & 1)) pr.push_back({perm[a], perm[a | (1 << J)]});
                for (size_t q = 0; q < pr.size(); ++q) o << "      v4f r" << q << " = {0.f, 0.f, 0.f, 0.f};\n";
                for (int k = 0; k < 4; ++k)
                    for (size_t q = 0; q < pr.size(); ++q)
                        o << "      r" << q << " = __builtin_amdgcn_mfma_f32_4x4x1f32(w[" << k << "], x"
                          << (k < 2 ? pr[q].first : pr[q].second) << (k & 1 ? ".y" : ".x") << ", r" << q << ", 0, 0, 0);\n";
                for (size_t q = 0; q < pr.size(); ++q)
                    o << "      x" << pr[q].first << " = make_float2(r" << q << "[0], r" << q << "[1]); x" << pr[q].second
                      << " = make_float2(r" << q << "[2], r" << q << "[3]);\n";
                o << "    }\n";
                continue;
            }
            // Generic class: the outer controls decide per tile; fast classes have none.
            const bool outer = cls >= kFwdGenericClass && op.omask != 0;
            const bool lane_pred = cls >= 3 && tm != 0;
            const bool cond = lane_pred || outer;
            double uv[8];
            record_entries(op, c64, uv);
            const PairUpdate pu = pair_update(op.type, MK, uv, !bound[prog.pass_op0[p] + oi]);
            o << "    {\n";
            if (!pu.entries.empty()) o << "      const " << R << "* u = um + " << oi * UM << ";\n";
            if (cond) {
                o << "      const bool pc = true";
                if (lane_pred) o << " && ((ethr & " << tm << "u) == " << (op.cval & tm) << "u)";
                if (outer) o << " && ((base & " << U(op.omask) << ") == " << U(op.oval) << ")";
                o << ";\n";
                if (pu.neg) o << "      const unsigned sm = pc ? 0x80000000u : 0u;\n";
            }
            for (int a = 0; a < N; ++a) {
                if ((a >> J) & 1) continue;
                if (cls >= 3 && (er[a] & rm) != (op.cval & rm)) continue;
                if (op.type == OT_SWAP && !cond) {
                    std::swap(perm[a], perm[a | (1 << J)]);
                    continue;
                }
                o << pair_code(pu, V, "x" + I(perm[a]), "x" + I(perm[a | (1 << J)]), cond);
            }
            o << "    }\n";
        }
        for (int r = 0; r < N; ++r) o << "    " << at("sw", er[r]) << " = x" << perm[r] << ";\n";
        o << "  }\n  __syncthreads();\n";
    }
    // Store: element e = th + r * nthr of the stored tile comes from LDS tile element
    // sth | sreg[r], thread bit i moving to tile bit store_src[i].
    for (int k = 0; k < t - RB; ++k) thread_bits[k] = pass.store_src.empty() ? k : pass.store_src[k];
    o << "  " << thread_position("ssw", thread_bits) << "  ssw *= " << es << "u;\n";
    if (P.B > 1) o << "  if (b0 + bl < " << P.B << "u) {\n";
    for (int r = 0; r < N; ++r) {
        uint32_t v = 0;
        for (int j = 0; j < RB; ++j)
            if ((r >> j) & 1) v |= 1u << (pass.store_src.empty() ? t - RB + j : pass.store_src[t - RB + j]);
        o << "  gp[toff + " << U(rofs[r]) << "] = " << at("ssw", v) << ";\n";
    }
    if (P.B > 1) o << "  }\n";
    o << "}\n";
    *nthr_out = nthr;
    *lds_out = lds;
    return o.str();
}

// Gradient term of one pair for generator class gen (Re or Im of lambda^dagger M psi on the
// pair, the generic kernels' formulas): p0, p1 psi and l0, l1 lambda of the pair.
std::string grad_expr(int gen, const std::string& p0, const std::string& p1, const std::string& l0,
                      const std::string& l1)
{
    switch (gen) {
    case GEN_X: return "fma(" + l0 + ".x, " + p1 + ".y, fma(-" + l0 + ".y, " + p1 + ".x, fma(" + l1 + ".x, " + p0 + ".y, -" + l1 + ".y * " + p0 + ".x)))";
    case GEN_Y: return "fma(" + l1 + ".x, " + p0 + ".x, fma(" + l1 + ".y, " + p0 + ".y, fma(-" + l0 + ".x, " + p1 + ".x, -" + l0 + ".y * " + p1 + ".y)))";
    case GEN_Z: return "fma(" + l0 + ".x, " + p0 + ".y, fma(-" + l0 + ".y, " + p0 + ".x, fma(-" + l1 + ".x, " + p1 + ".y, " + l1 + ".y * " + p1 + ".x)))";
    case GEN_P1: return "(-2.0 * fma(" + l1 + ".x, " + p1 + ".y, -" + l1 + ".y * " + p1 + ".x))";
    default:
        return "dense_grad(gm, " + p0 + ", " + p1 + ", " + l0 + ", " + l1 + ")";
    }
}

const char* kBwdPrelude = R"YAO(
template <int CTRL> __device__ __forceinline__ double dpp_f64(double v)
{
    const u64 b = __builtin_bit_cast(u64, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)b, CTRL, 0xF, 0xF, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((u64)hi << 32) | lo);
}
// Sum over the lanes of a 16-lane DPP row that share their low C bits (a batch slot): lanes 0 .. 2^C - 1
// of the row hold them.
template <int C> __device__ __forceinline__ double row_sum16(double v)
{
    if (C < 1) v += dpp_f64<0xB1>(v);
    if (C < 2) v += dpp_f64<0x4E>(v);
    if (C < 3) v += dpp_f64<0x124>(v);
    v += dpp_f64<0x128>(v);
    return v;
}
// The unit forms of rotations about X and Z on a pair.
__device__ __forceinline__ void rx_unit(double2& a, double2& b, double k)
{
    const double2 p = a, q = b;
    a = make_double2(fma(-k, q.y, p.x), fma(k, q.x, p.y));
    b = make_double2(fma(-k, p.y, q.x), fma(k, p.x, q.y));
}
__device__ __forceinline__ void rz_unit(double2& a, double2& b, double k)
{
    const double2 p = a, q = b;
    a = make_double2(fma(-k, p.y, p.x), fma(k, p.x, p.y));
    b = make_double2(fma(k, q.y, q.x), fma(-k, q.x, q.y));
}
// |F| < 2^-40 (the high word of F below lim), wave-uniform.
constexpr unsigned kScaleLow = (1023u - 40u) << 20;
__device__ __forceinline__ bool scale_low(double F, unsigned lim)
{
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(__builtin_bit_cast(u64, F) >> 32));
    return (hi & 0x7fffffffu) < lim;
}
// Exchanges two double2 registers in place (v_swap_b32 on each 32-bit half), so that a swap
// under a lane mask needs neither selects nor copies where the lanes rejoin.
__device__ __forceinline__ void swap_d2(double2& a, double2& b)
{
    unsigned* x = reinterpret_cast<unsigned*>(&a);
    unsigned* y = reinterpret_cast<unsigned*>(&b);
    asm volatile("v_swap_b32 %0, %1\n\tv_swap_b32 %2, %3\n\tv_swap_b32 %4, %5\n\tv_swap_b32 %6, %7"
                 : "+v"(x[0]), "+v"(y[0]), "+v"(x[1]), "+v"(y[1]), "+v"(x[2]), "+v"(y[2]), "+v"(x[3]), "+v"(y[3]));
}
// 2 Re(conj(l) M p) for a dense 2 x 2 generator M (re[4], im[4], row-major).
__device__ __forceinline__ double dense_grad(const CST double* m, double2 p0, double2 p1, double2 l0, double2 l1)
{
    const double m0x = m[0] * p0.x - m[4] * p0.y + m[1] * p1.x - m[5] * p1.y;
    const double m0y = m[0] * p0.y + m[4] * p0.x + m[1] * p1.y + m[5] * p1.x;
    const double m1x = m[2] * p0.x - m[6] * p0.y + m[3] * p1.x - m[7] * p1.y;
    const double m1y = m[2] * p0.y + m[6] * p0.x + m[3] * p1.y + m[7] * p1.x;
    return 2.0 * (l0.x * m0x + l0.y * m0y + l1.x * m1x + l1.y * m1y);
}
)YAO";

// Code of one reverse pass (psi in FP64, lambda in the state's precision), or an empty
// string when the pass is not supported.
std::string gen_backward_pass(const Plan& P, const Program& prog, int p, int n, int dtype, const std::string& name,
                              int* nthr_out, size_t* lds_out)
{
    const HostPass& pass = P.passes[p];
    const int RB = P.reg_bits, N = 1 << RB, t = P.t;
    if (pass.standalone >= 0) return "";
    if (t - RB < 4 || t - RB > 10 || (int)pass.tile_qubits.size() != t - P.c) return "";
    const int g0 = prog.pass_group0[p], ng = (int)pass.groups.size();
    int maxslots = 0;
    for (int g = 0; g < ng; ++g) {
        if (prog.groups[g0 + g].lds) return "";
        maxslots = std::max(maxslots, prog.groups[g0 + g].nslot);
    }
    const bool c64 = dtype == YAO_C64;
    const int nthr = 1 << (t - RB);
    const int lb = c64 ? 8 : 16;
    // Gradient partials: each gradient is summed over lane pairs (one DPP step; lanes 8 apart in a
    // batch, whose slots are the low c <= 3 lane bits) and the pair sums go to LDS, E = nthr / 2
    // entries per gradient, two buffers of the group's gradients; when that does not fit, per slot
    // over rows of 16 lanes (E = 2^c nthr / 16).
    auto lds_for = [&](int e) {
        return ((size_t)(16 + lb) << t) + sizeof(double) * 2 * (size_t)std::max(1, maxslots) * e;
    };
    const int red_lanes = lds_for(nthr >> 1) <= 160 * 1024 ? 2 : 16;
    const int E = red_lanes == 2 ? nthr / 2 : (nthr / 16) << P.c;
    const size_t lds = lds_for(E);
    if (lds > 160 * 1024) return "";
    const std::string VL = c64 ? "float2" : "double2", RL = c64 ? "float" : "double";
    std::ostringstream o;
    // Workgroups per CU that the LDS allows; when that is more than the registers would
    // allow at the compiler's choice, ask for the register budget that fits them.
    const int wg_lds = (int)std::min<size_t>(8, (160 * 1024) / lds);
    const int waves = std::max(1, wg_lds * (nthr / 64) / 4);  // per SIMD
    o << "extern \"C\" __global__ void __launch_bounds__(" << nthr << ") __attribute__((amdgpu_waves_per_eu("
      << std::min(waves, 8) << "))) " << name
      << "(void* psi_, void* lam_, const char* ops_, const double* mats, double* gpart_, const char* zs_, int op_first, "
         "int pstride) {\n";
    o << "  __shared__ __align__(16) unsigned char smem[" << lds << "];\n";
    // Lambda, psi, partials, in this order: the first two within the offsets of an LDS instruction.
    // Positions are kept in units of 8 bytes' lambda (or 16 bytes') and psi's by a factor, one XOR an access.
    auto at_psi = [&](const std::string& pos, uint32_t e) {
        return "*(LDS double2*)((LDS char*)smem + " + I((long long)lb << t) + " + (" + pos + "p ^ " + I((long long)swz_host(e) * 16) + "u))";
    };
    auto at_lam = [&](const std::string& pos, uint32_t e) {
        return "*(LDS " + VL + "*)((LDS char*)smem + (" + pos + "l ^ " + I((long long)swz_host(e) * lb) + "u))";
    };
    auto positions = [&](const std::string& name, const std::vector<int>& bits) {
        return thread_position(name, bits) + "    const unsigned " + name + "p = " + name + " * 16u, " + name + "l = " + name +
               " * " + I(lb) + "u;\n";
    };
    std::vector<int> thread_bits(t - RB);
    for (int k = 0; k < t - RB; ++k) thread_bits[k] = k;
    o << "  double* red0 = (double*)(smem + " << ((16 + lb) << t) << ");\n";
    o << "  const unsigned th = threadIdx.x;\n";
    o << "  GLB double2* gp = (GLB double2*)psi_;\n  GLB " << VL << "* gl = (GLB " << VL << "*)lam_;\n";
    o << "  const CST char* ops = (const CST char*)ops_;\n  GLB double* gpart = (GLB double*)gpart_;\n";
    o << "  if (zs_) { const CST u64* z = (const CST u64*)(zs_ + 32 * blockIdx.z); gp = (GLB double2*)z[0]; gl = (GLB "
      << VL << "*)z[1]; ops = (const CST char*)z[2] + (u64)op_first * " << sizeof(POp)
      << "; gpart = (GLB double*)z[3]; }\n";
    std::vector<uint64_t> rofs;
    o << tile_code(P, pass, n, rofs);
    o << "  {\n";
    // Lambda of complex64 states as 64-bit words (as two floats, which the maximum below reads, its writes to LDS
    // come out as pairs of 32 bits).
    const std::string WL = c64 ? "u64" : VL;
    for (int r = 0; r < N; ++r)
        o << "    const double2 v" << r << " = gp[toff + " << U(rofs[r]) << "]; const " << WL << " w" << r << " = ((GLB " << WL
          << "*)gl)[toff + " << U(rofs[r]) << "];\n";
    o << "    " << positions("lpos", thread_bits);
    for (int r = 0; r < N; ++r)
        o << "    " << at_psi("lpos", (uint32_t)r * nthr) << " = v" << r << "; *(LDS " << WL << "*)&"
          << at_lam("lpos", (uint32_t)r * nthr) << " = w" << r << ";\n";
    // big: some lambda of the tile is at 2^80 or above (see the scale F below). A word a wave, in the second
    // buffer of partials, which the second register group writes first.
    const size_t big_at = ((size_t)(16 + lb) << t) + sizeof(double) * (size_t)std::max(1, maxslots) * E;
    if (c64) {
        o << "    unsigned wm = 0;\n";
        for (int r = 0; r < N; ++r)
            o << "    wm = max(wm, max((unsigned)w" << r << " & 0x7fffffffu, (unsigned)(w" << r << " >> 32) & 0x7fffffffu));\n";
        o << "    const u64 wide = __builtin_amdgcn_ballot_w64(wm >= " << ((127 + 80) << 23) << "u);\n"
          << "    ((LDS unsigned*)((LDS char*)smem + " << big_at << "))[th >> 6] = wide != 0;\n";  // every lane the same
    }
    o << "  }\n  __syncthreads();\n";
    o << "  double F = 1.0;\n";
    if (c64) {
        o << "  unsigned big = 0;\n";
        for (int i = 0; i < std::max(1, nthr / 64); ++i)
            o << "  big |= ((LDS unsigned*)((LDS char*)smem + " << big_at << "))[" << i << "];\n";
        o << "  const unsigned lim = __builtin_amdgcn_readfirstlane(big) ? 0xffffffffu : kScaleLow;\n";
    }
    // LDS address of a lane pair's first partial, kept in a register: the partials' own offsets are immediates.
    if (red_lanes == 2)
        o << "  unsigned rad = (unsigned)(u64)(LDS double*)red0 + " << (P.c ? "((th >> 4) * 8u + (th & 7u))" : "(th >> 1)") << " * 8u;\n  asm volatile(\"\" : \"+v\"(rad));\n";
    // Matrix entries each op reads (cls 0 and 1: k and f as u1, u2;
    // others what their class needs). They come through the scalar cache a batch ahead:
    // batches of up to 8 consecutive ops (at most 16 entries); at the first op of batch b the
    // kernel waits for batch b's loads and issues batch b + 1's, so records that miss the
    // scalar cache are fetched while batch b computes. The loads are volatile so that the
    // compiler keeps them where they are issued instead of next to their uses.
    std::vector<std::pair<int, int>> seq;  // (group, op within group) in pass order
    for (int g = 0; g < ng; ++g)
        for (int i = 0; i < prog.groups[g0 + g].nops; ++i) seq.push_back({g, i});
    const std::vector<char> bound = bound_ops(prog);
    auto reverse_update = [&](int oi) {
        const POp& op = prog.ops[prog.pass_op0[p] + oi];
        return pair_update(op.type, "make_double2", op.u, !bound[prog.pass_op0[p] + oi]);
    };
    auto coeffs = [&](int oi) -> std::vector<int> {
        const int cls = prog.ops[prog.pass_op0[p] + oi].var / RB;
        if (cls <= 1) return {1, 2};
        return reverse_update(oi).entries;
    };
    auto op_index = [&](size_t i) { return prog.groups[g0 + seq[i].first].op0 + seq[i].second; };
    std::vector<size_t> batch_first;  // first op (in seq) of each batch
    {
        int cnt = 0, ent = 0;
        for (size_t i = 0; i < seq.size(); ++i) {
            const int c = (int)coeffs(op_index(i)).size();
            if (batch_first.empty() || cnt == 8 || ent + c > 16) {
                batch_first.push_back(i);
                cnt = 0;
                ent = 0;
            }
            ++cnt;
            ent += c;
        }
        batch_first.push_back(seq.size());
    }
    auto emit_loads = [&](size_t b) {
        if (b + 1 >= batch_first.size()) return;
        for (size_t i = batch_first[b]; i < batch_first[b + 1]; ++i)
            for (int k : coeffs(op_index(i)))
                o << "    U" << i << "_" << k << " = ((const volatile CST double*)(ops + "
                  << (size_t)op_index(i) * sizeof(POp) + offsetof(POp, u) << "))[" << k << "];\n";
    };
    for (size_t i = 0; i < seq.size(); ++i)
        for (int k : coeffs(op_index(i))) o << "  double U" << i << "_" << k << ";\n";
    // Rotations run in their unit form (split_rotation): an update takes one FMA per real number where
    // the plain matrix takes a multiply and an FMA, and their factors f collect in F, common to psi,
    // lambda and every element (gradients take F^2). The values in registers are 1 / F of what they
    // stand for; where |F| has come below 2^-40 they are multiplied by it, looked at after every
    // kScaledOps rotations and before lambda is rounded to the state's precision at a group's end. Range:
    // the cosine of half of pi is 2^-54 in FP64 and no finite angle's is below 2^-61, so the F that a gradient
    // takes has at most five such factors and stays above 2^-345, F^2 above 2^-690; the products of two
    // values in registers stay finite for |psi| |lambda| up to 2^334 (looked at after eight rotations: 2^90).
    // Lambda lies in LDS as float for complex64 states, up to 2^40 above its value: tiles with an entry over
    // 2^80 (their norm, and so every later entry, is below 2^86 where there is none) multiply by F at
    // every group's end. FP64 issue is most of a reverse pass: with
    // 16 + 16 + 32 instructions for an Rx on 8 amplitudes in place of 16 + 64, with no phase
    // entries left among the scalar loads (they had spilled into vector lanes behind a wait each) and
    // the group's sums through DPP adds instead of LDS permutes, the 20-qubit depth-20 sweep's twelve
    // passes went from 737 to 636 us.
    constexpr int kScaledOps = 6;
    bool scaled = false;  // F may differ from 1
    int nscaled = 0;
    auto emit_rescale = [&](bool rounds) {
        o << "    if (scale_low(F, " << (rounds && c64 ? "lim" : "kScaleLow") << ")) {\n";
        for (int r = 0; r < N; ++r)
            o << "      x" << r << ".x *= F; x" << r << ".y *= F; y" << r << ".x *= F; y" << r << ".y *= F;\n";
        o << "      F = 1.0;\n    }\n";
        nscaled = 0;
    };
    size_t si = 0, bi = 0;
    emit_loads(0);
    int buf = 0;
    for (int g = 0; g < ng; ++g) {
        const PGroupDesc& G = prog.groups[g0 + g];
        uint32_t rmask = 0;
        for (int j = 0; j < RB; ++j) rmask |= 1u << G.rpos[j];
        std::vector<uint32_t> er(N);
        for (int r = 0; r < N; ++r) {
            uint32_t e = 0;
            for (int j = 0; j < RB; ++j)
                if ((r >> j) & 1) e |= 1u << G.rpos[j];
            er[r] = e;
        }
        const std::vector<int> lanes = lane_order(t, P.c, rmask);
        o << "  {\n    unsigned ethr = 0;\n";
        for (size_t k = 0; k < lanes.size(); ++k) o << "    ethr |= ((th >> " << k << ") & 1u) << " << lanes[k] << ";\n";
        o << "    " << positions("sw", lanes);
        if (red_lanes != 2) o << "    double* red = red0 + " << buf * std::max(1, maxslots) * E << ";\n";
        std::vector<int> perm(N);
        for (int r = 0; r < N; ++r) {
            perm[r] = r;
            o << "    double2 x" << r << " = " << at_psi("sw", er[r]) << "; double2 y" << r << "; { const " << VL << " q = "
              << at_lam("sw", er[r]) << "; y" << r << " = make_double2((double)q.x, (double)q.y); }\n";
        }
        int nslot = 0;
        for (int i = 0; i < G.nops; ++i) {
            const int oi = G.op0 + i;
            const POp& op = prog.ops[prog.pass_op0[p] + oi];
            const int J = op.rpos;
            const int cls = op.var / RB;
            const uint32_t tm = op.cmask & ~rmask, rm = op.cmask & rmask;
            const bool generic = cls >= kBwdGenericClass;
            const bool outer = generic && op.omask != 0;
            const bool lane_pred = (cls == 2 || generic) && tm != 0;
            const bool cond = lane_pred || outer;
            // Reverse ops read their matrices through the scalar cache (in LDS they would occupy
            // VGPRs, and the reverse kernel has none to spare), prefetched one op ahead.
            if (si == batch_first[bi]) {
                o << "    __builtin_amdgcn_s_waitcnt(0xC07F);\n    __builtin_amdgcn_sched_barrier(0);\n";
                emit_loads(++bi);
                o << "    __builtin_amdgcn_sched_barrier(0);\n";
            }
            const size_t cur = si++;
            const PairUpdate pu = reverse_update(oi);
            std::ostringstream enclosing;
            std::swap(o, enclosing);  // the op's code goes to its own stream first
            o << "    {\n";
            if (generic && op.slot >= 0 && op.gen == GEN_DENSE)
                o << "      const CST double* gm = (const CST double*)mats + " << op.mat + 8 << ";\n";
            if (cond) {
                o << "      const bool pc = true";
                if (lane_pred) o << " && ((ethr & " << tm << "u) == " << (op.cval & tm) << "u)";
                if (outer) o << " && ((base & " << U(op.omask) << ") == " << U(op.oval) << ")";
                o << ";\n";
                if (pu.neg) o << "      const unsigned sm = pc ? 0x80000000u : 0u;\n";
            }
            // Pairs whose register-bit controls hold.
            std::vector<int> pairs;
            for (int a = 0; a < N; ++a) {
                if ((a >> J) & 1) continue;
                if ((cls == 2 || generic) && (er[a] & rm) != (op.cval & rm)) continue;
                pairs.push_back(a);
            }
            // Gradient from psi and lambda before the update (both are 1 / F of what they stand for).
            if (op.slot >= 0) {
                const int gen = cls == 0 ? GEN_X : cls == 1 ? GEN_Z : op.gen;
                o << "      double g" << (pairs.empty() || cond ? " = 0.0" : "") << ";\n";
                for (int a : pairs) {
                    const std::string e = grad_expr(gen, "x" + I(perm[a]), "x" + I(perm[a | (1 << J)]), "y" + I(perm[a]),
                                                    "y" + I(perm[a | (1 << J)]));
                    if (cond) o << "      g += pc ? " << e << " : 0.0;\n";
                    else o << "      g " << (a == pairs.front() ? "= " : "+= ") << e << ";\n";
                }
                if (scaled) o << "      g *= F * F;\n";
                if (red_lanes == 2)  // both lanes of a pair hold the sum and write it
                    o << "      g += dpp_f64<" << (P.c ? "0x128" : "0xB1") << ">(g);\n      *(LDS double*)(rad + " << (buf * std::max(1, maxslots) + nslot) * E * 8
                      << "u) = g;\n";
                else
                    o << "      g = row_sum16<" << P.c << ">(g);\n      if ((th & 15u) < " << (1 << P.c) << "u) red[" << nslot * E
                      << " + ((th >> 4) << " << P.c << ") + (th & 15u)] = g;\n";
                ++nslot;
            }
            for (int a : pairs) {
                const std::string X = "x" + I(perm[a]), Y = "x" + I(perm[a | (1 << J)]);
                const std::string LX = "y" + I(perm[a]), LY = "y" + I(perm[a | (1 << J)]);
                if (op.type == OT_SWAP && (cls == 2 || !cond)) {
                    if (!cond) {
                        std::swap(perm[a], perm[a | (1 << J)]);
                    } else {
                        // Swapped in place under the lane mask: one branch around the op's pairs,
                        // no selects and no copies where the lanes rejoin.
                        if (a == pairs.front()) o << "      if (pc) {\n";
                        o << "        swap_d2(" << X << ", " << Y << "); swap_d2(" << LX << ", " << LY << ");\n";
                        if (a == pairs.back()) o << "      }\n";
                    }
                    continue;
                }
                for (const auto& pr : {std::make_pair(X, Y), std::make_pair(LX, LY)}) {
                    const std::string& A = pr.first;
                    const std::string& B = pr.second;
                    if (cls == 0) {  // f (a + i k b, i k a + b)
                        o << "      rx_unit(" << A << ", " << B << ", u[1]);\n";
                    } else if (cls == 1) {  // f (a + i k a, b - i k b)
                        o << "      rz_unit(" << A << ", " << B << ", u[1]);\n";
                    } else {
                        o << pair_code(pu, "double2", A, B, cond);
                    }
                }
            }
            if (cls <= 1) {
                o << "      F *= u[2];\n";
                scaled = true;
                if (++nscaled == kScaledOps) emit_rescale(false);
            }
            o << "    }\n";
            // The op's u[k] are the prefetched U<cur>_k.
            std::string body = o.str();
            for (int k = 0; k < 8; ++k) {
                const std::string from = "u[" + I(k) + "]", to = "U" + I((long long)cur) + "_" + I(k);
                for (size_t pos = body.find(from); pos != std::string::npos; pos = body.find(from, pos + to.size()))
                    body.replace(pos, from.size(), to);
            }
            std::swap(o, enclosing);
            o << body;
        }
        if (nslot != G.nslot) return "";  // the record's slots and the group's list disagree
        if (scaled) emit_rescale(true);
        for (int r = 0; r < N; ++r)
            o << "    " << at_psi("sw", er[r]) << " = x" << perm[r] << "; " << at_lam("sw", er[r]) << " = make_"
              << VL << "((" << RL << ")y" << perm[r] << ".x, (" << RL << ")y" << perm[r] << ".y);\n";
        o << "  }\n  __syncthreads();\n";
        if (nslot > 0) {
            // Partials of each gradient over the tile: 16 tasks per gradient, E entries each.
            o << "  {\n    const double* red = red0 + " << buf * std::max(1, maxslots) * E << ";\n";
            o << "    for (unsigned task = th; task < " << nslot * 16 << "u; task += " << nthr << "u) {\n";
            o << "      const unsigned s = task >> 4, j = task & 15u;\n      double v = 0.0;\n";
            o << "      for (unsigned e = j; e < " << E << "u; e += 16u) v += red[s * " << E << "u + e];\n";
            o << "      v = row_sum16<" << P.c << ">(v);\n";  // the 16 lanes of a task are one DPP row
            o << "      int slot = " << G.slots[0] << ";\n";
            for (int k = 1; k < nslot; ++k) o << "      if (s == " << k << "u) slot = " << G.slots[k] << ";\n";
            if (P.B == 1) o << "      if (j == 0) gpart[(u64)slot * (u64)pstride + blockIdx.x] = v;\n    }\n  }\n";
            else
                o << "      if (j < " << (1 << P.c) << "u && b0 + j < " << P.B << "u) gpart[((u64)slot * " << P.B
                  << "ull + b0 + j) * (u64)pstride + blockIdx.x] = v;\n    }\n  }\n";
            buf ^= 1;
        }
    }
    // Store with the accumulated scale.
    for (int k = 0; k < t - RB; ++k) thread_bits[k] = pass.store_src.empty() ? k : pass.store_src[k];
    o << "  " << positions("ssw", thread_bits);
    if (P.B > 1) o << "  if (b0 + bl < " << P.B << "u) {\n";
    for (int r = 0; r < N; ++r) {
        uint32_t v = 0;
        for (int j = 0; j < RB; ++j)
            if ((r >> j) & 1) v |= 1u << (pass.store_src.empty() ? t - RB + j : pass.store_src[t - RB + j]);
        o << "  { const double2 v = " << at_psi("ssw", v) << "; const " << VL << " w = " << at_lam("ssw", v)
          << "; const double wx = (double)w.x, wy = (double)w.y;\n";
        o << "    gp[toff + " << U(rofs[r]) << "] = make_double2(F * v.x, F * v.y);\n";
        o << "    gl[toff + " << U(rofs[r]) << "] = make_" << VL << "((" << RL << ")(F * wx), (" << RL << ")(F * wy)); }\n";
    }
    if (P.B > 1) o << "  }\n";
    o << "}\n";
    *nthr_out = nthr;
    *lds_out = lds;
    return o.str();
}

std::mutex g_jit_mu;
int g_suspend = 0;
std::atomic<long long> g_compiled_programs{0}, g_compiled_passes{0}, g_failures{0};
std::atomic<long long> g_launches_fwd{0}, g_launches_bwd{0};

// A program that could not be compiled keeps the generic kernels; say why, once per program.
void report_failure(const char* what, const std::string& detail)
{
    ++g_failures;
    fprintf(stderr, "yao: run-time compiled passes unavailable (%s): %.300s; using the generic kernels\n", what,
            detail.c_str());
}

}  // namespace

bool takes_real_form(const Plan& P, const POp& op)
{
    // Whole waves; class 2: dense without controls.
    return P.compiled && P.t - P.reg_bits >= 6 && op.k == 1 && op.var / P.reg_bits == 2;
}

void use_real_forms(const Plan& P, Program& prog)
{
    std::vector<char> bound = bound_ops(prog);
    for (size_t i = 0; i < prog.ops.size(); ++i) {
        POp& op = prog.ops[i];
        if (!takes_real_form(P, op) || bound[i]) continue;
        const double* m = prog.mats.data() + op.mat;  // the pool keeps the FP64 entries: re[4], im[4]
        real_form(m, m + 4, (float*)op.u);
    }
    for (BindRec& b : prog.binds)
        if (takes_real_form(P, prog.ops[b.op])) b.mode = 5;
}

struct JitPasses {
    std::vector<hipModule_t> mod;   // per pass
    std::vector<hipFunction_t> fn;  // per pass; null: the generic kernel
    std::vector<int> nthr;
    std::vector<size_t> lds;
    std::vector<int> ntiles, nslots;  // grid x and y
};

void jit_suspend(bool on)
{
    std::lock_guard<std::mutex> lk(g_jit_mu);
    g_suspend += on ? 1 : -1;
}

namespace {

// Source of each supported pass of a program (empty for passes left to the generic kernel),
// every pass a program of its own so that the passes compile in parallel.
int jit_source(const Plan& P, const Program& prog, bool bwd, int dtype, int n, std::vector<std::string>& src,
               std::vector<int>& nthr, std::vector<size_t>& lds)
{
    src.assign(P.passes.size(), "");
    nthr.assign(P.passes.size(), 0);
    lds.assign(P.passes.size(), 0);
    int count = 0;
    for (size_t p = 0; p < P.passes.size(); ++p) {
        const std::string code = bwd ? gen_backward_pass(P, prog, (int)p, n, dtype, "yao_pass_bwd", &nthr[p], &lds[p])
                                     : gen_forward_pass(P, prog, (int)p, n, dtype, "yao_pass_fwd", &nthr[p], &lds[p]);
        if (code.empty()) continue;
        src[p] = std::string(kPrelude) + (bwd ? kBwdPrelude : "") + code;
        ++count;
    }
    return count;
}

// Compile the non-empty sources on a few host threads; code[p] stays empty for a failure, and
// logs[p] then holds the compiler log.
std::vector<char> jit_build(const std::string& src, std::string* log);
void jit_build_all(const std::vector<std::string>& src, std::vector<std::vector<char>>& code,
                   std::vector<std::string>& logs)
{
    code.assign(src.size(), {});
    logs.assign(src.size(), "");
    std::atomic<size_t> next{0};
    auto work = [&] {
        for (size_t p; (p = next.fetch_add(1)) < src.size();)
            if (!src[p].empty()) code[p] = jit_build(src[p], &logs[p]);
    };
    const unsigned hw = std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
    std::vector<std::thread> th;
    for (unsigned i = 1; i < hw && i < src.size(); ++i) th.emplace_back(work);
    work();
    for (std::thread& x : th) x.join();
}

// hipRTC compile for gfx950 with the library's own code-generation flags. Returns the code
// object, or an empty vector with the compiler log in *log.
std::vector<char> jit_build(const std::string& src, std::string* log)
{
    std::vector<char> code;
    hiprtcProgram rp;
    if (hiprtcCreateProgram(&rp, src.c_str(), "yao_pass.hip", 0, nullptr, nullptr) != HIPRTC_SUCCESS) {
        if (log) *log = "hiprtcCreateProgram failed";
        return code;
    }
    // The load/store vectorizer finds nothing to merge here (LDS rows are XOR-swizzled, tile
    // rows far apart) and costs a sixth of the compile time.
    const char* opts[] = {"--offload-arch=gfx950", "-O3", "-ffp-contract=fast", "-Xclang", "-target-feature",
                          "-Xclang", "-packed-fp32-ops", "-mllvm", "-amdgpu-load-store-vectorizer=false"};
    if (hiprtcCompileProgram(rp, (int)(sizeof(opts) / sizeof(opts[0])), opts) == HIPRTC_SUCCESS) {
        size_t cs = 0;
        if (hiprtcGetCodeSize(rp, &cs) == HIPRTC_SUCCESS && cs > 0) {
            code.resize(cs);
            if (hiprtcGetCode(rp, code.data()) != HIPRTC_SUCCESS) code.clear();
        }
    } else if (log) {
        size_t ls = 0;
        if (hiprtcGetProgramLogSize(rp, &ls) == HIPRTC_SUCCESS && ls > 0) {
            std::string l(ls, '\0');
            if (hiprtcGetProgramLog(rp, &l[0]) == HIPRTC_SUCCESS) *log = l;
        }
    }
    (void)hiprtcDestroyProgram(&rp);
    return code;
}

}  // namespace

// Compile every supported pass of a bound program into one module. Returns nullptr (and
// leaves the program on the generic kernels) when nothing is supported or compiling fails.
static JitPasses* jit_compile(const Plan& P, const Program& prog, bool bwd, int dtype, int n)
{
    std::vector<std::string> src, logs;
    std::vector<int> nthr;
    std::vector<size_t> lds;
    if (jit_source(P, prog, bwd, dtype, n, src, nthr, lds) == 0) return nullptr;
    std::vector<std::vector<char>> code;
    jit_build_all(src, code, logs);
    for (size_t p = 0; p < src.size(); ++p)
        if (!src[p].empty() && code[p].empty()) {
            report_failure("compile", logs[p]);
            return nullptr;
        }
    JitPasses* J = new JitPasses;
    J->mod.assign(P.passes.size(), nullptr);
    J->fn.assign(P.passes.size(), nullptr);
    J->nthr = nthr;
    J->lds = lds;
    J->ntiles.assign(P.passes.size(), 0);
    J->nslots.assign(P.passes.size(), 1);
    for (size_t p = 0; p < P.passes.size(); ++p) {
        if (code[p].empty()) continue;
        hipError_t e = hipModuleLoadData(&J->mod[p], code[p].data());
        if (e == hipSuccess) e = hipModuleGetFunction(&J->fn[p], J->mod[p], bwd ? "yao_pass_bwd" : "yao_pass_fwd");
        if (e != hipSuccess) {
            report_failure("module load", hipGetErrorString(e));
            jit_free(J);
            return nullptr;
        }
        J->ntiles[p] = 1 << (n - (P.t - P.c));
        J->nslots[p] = (P.B + (1 << P.c) - 1) >> P.c;
        ++g_compiled_passes;
    }
    ++g_compiled_programs;
    return J;
}

const JitPasses* jit_passes(const BoundProgram* bp, const Plan& P, bool bwd, int dtype, int n, int B)
{
    if (!bp || B != P.B) return nullptr;
    const int when = options().jit;
    std::lock_guard<std::mutex> lk(g_jit_mu);
    if (bp->jit || bp->jit_failed) return bp->jit;
    if (when <= 0 || g_suspend > 0 || recording()) return nullptr;
    if (++bp->uses < when) return nullptr;
    bp->jit = jit_compile(P, bp->prog, bwd, dtype, n);
    if (!bp->jit) bp->jit_failed = true;
    return bp->jit;
}

bool jit_due(const BoundProgram* bp)
{
    if (!bp) return false;
    const int when = options().jit;
    std::lock_guard<std::mutex> lk(g_jit_mu);
    if (bp->alt) return true;
    if (when <= 0 || g_suspend > 0 || recording()) return false;
    return ++bp->alt_uses >= when;
}

bool jit_compile_all(const BoundProgram* bp, const Plan& P, bool bwd, int dtype, int n)
{
    std::lock_guard<std::mutex> lk(g_jit_mu);
    if (!bp->jit && !bp->jit_failed) {
        std::vector<std::string> src;
        std::vector<int> nthr;
        std::vector<size_t> lds;
        if (jit_source(P, bp->prog, bwd, dtype, n, src, nthr, lds) == (int)P.passes.size())
            bp->jit = jit_compile(P, bp->prog, bwd, dtype, n);
        if (!bp->jit) bp->jit_failed = true;
    }
    return bp->jit != nullptr;
}

// Sizes of compiled plans, from sweeps over tile and register bits. Times are of all passes of one
// sweep of the layered ansatz, in us.
//
// Reverse: a pass takes as long for one tile as for a tile on every CU, so while 2^10-element tiles
// leave CUs idle they win over 2^12 although they take more passes (15 qubits, depth 10,
// complex64: 131 in 6 passes against 196 in 4; 17 qubits: 197 / 283; 18 qubits: 222 / 297; 14 qubits
// complex128: 126 / 140), and with 4 elements a thread a tile still has a wave on every SIMD (8
// elements: 17 qubits 235; 2^11 tiles: 225). At 20 qubits the vector units are busy and the larger
// tile's fewer passes win (636 against 724 for 2^11 and 795 for 2^10); 19 qubits lie between
// (complex64: 2^10 320, 2^11 269, 2^12 359; complex128: 253, 276).
//
// Forward: 8 elements a thread give two waves per SIMD where 16 give one (20 qubits complex64: 237
// against 291; 10 qubits complex128: 19 against 25). Above 20 qubits several tiles share a CU and
// 16 elements, with fewer exchanges through LDS, win (24 qubits complex64: 708 against 744).
// Batches keep the generic sizes (20 qubits, 64 slots, depth 20: reverse passes 39.6 ms in 2^12 tiles,
// 41.1 in 2^11; with the generic kernels 74 ms) but for small ones (10 qubits, 100 slots: 63 / 80).
// Complex128 tiles of 2^10 win up to 18 qubits (14 qubits: 68 against 95; 18 qubits: 110 / 143).
bool jit_geometry(int n, int B, int dtype, bool bwd, int* t, int* reg_bits, int* L)
{
    *L = dtype == YAO_C64 ? 4 : 3;
    if (B > 1) {
        *L = std::max(0, *L - std::min(3, ilog2_ceil((uint64_t)B)));
        if (!bwd) return dtype == YAO_C64;
        *t = std::min(*t, 11);
        return dtype == YAO_C64 && n + ilog2_ceil((uint64_t)B) <= 18;
    }
    if (bwd) {
        if (n > 19) return false;
        const bool mid = n == 19 && dtype == YAO_C64;
        *t = mid ? 11 : std::min(n, 10);
        *reg_bits = mid ? 3 : n >= 8 ? 2 : 1;
        return true;
    }
    if (n > 20) return dtype == YAO_C64;  // the generic kernels' sizes, records in real form
    const bool small = dtype == YAO_C128 && n > 12 && n <= 18;
    *t = std::min(n, small ? 10 : 12);
    *reg_bits = small || n <= 8 ? 2 : 3;
    return true;
}

bool jit_has(const JitPasses* J, int p)
{
    return J && p < (int)J->fn.size() && J->fn[p];
}

int jit_launch_forward(const JitPasses* J, int p, void* psi, const POp* ops, int op_first, double bytes,
                       double flops)
{
    const ZSlot* zs = zbatch_slots();
    const int nz = zs ? zbatch_count() : 1;
    struct {
        void* psi;
        const void* ops;
        const void* zs;
        int op_first;
        int pad;
    } args{psi, ops + op_first, zs, op_first, 0};
    size_t asz = sizeof(args);
    void* cfg[] = {HIP_LAUNCH_PARAM_BUFFER_POINTER, &args, HIP_LAUNCH_PARAM_BUFFER_SIZE, &asz, HIP_LAUNCH_PARAM_END};
    ++g_launches_fwd;
    const int pi = prof_begin(YAO_KF_PASS_FWD);
    YAO_HIP(hipModuleLaunchKernel(J->fn[p], (unsigned)J->ntiles[p], (unsigned)J->nslots[p], (unsigned)nz, (unsigned)J->nthr[p], 1, 1, 0,
                                  stream(), nullptr, cfg));
    prof_end(pi, bytes * nz, flops * nz);
    return 0;
}

int jit_selfcheck(const yao_circuit* c, int dtype, int reverse, int tile_qubits, int* npasses, int* njit)
{
    const int n = c->n;
    const bool bwd = reverse != 0;
    int t, cb, L;
    tile_geometry_tq(n, 1, dtype, bwd, tile_qubits, &t, &cb, &L);
    if (t - cb < kMaxRegBits + 1) return set_error(YAO_EINVAL, "circuit too small for tile passes");
    Plan P = get_plan(c, 0, (int)c->gates.size(), 1, t, cb, L, bwd, dtype == YAO_C64 ? 8 : 16);
    if (!P.valid) return set_error(YAO_EINVAL, "pass plan could not restore the qubit layout");
    P.compiled = true;
    Program prog;
    YAO_TRY(build_program(P, c, nullptr, bwd, dtype, prog));
    if (!prog.bindable) return set_error(YAO_EINVAL, "circuit cannot be bound on the device");
    if (!bwd && dtype == YAO_C64) use_real_forms(P, prog);
    std::vector<std::string> src, logs;
    std::vector<int> nthr;
    std::vector<size_t> lds;
    *npasses = (int)P.passes.size();
    *njit = jit_source(P, prog, bwd, dtype, n, src, nthr, lds);
    std::vector<std::vector<char>> code;
    jit_build_all(src, code, logs);
    for (size_t p = 0; p < src.size(); ++p)
        if (!src[p].empty() && code[p].empty())
            return set_error(YAO_EHIP, "run-time compile of pass %zu failed: %.400s", p, logs[p].c_str());
    return 0;
}

int jit_launch_backward(const JitPasses* J, int p, double* psi, void* lam, const POp* ops, int op_first,
                        const double* mats, double* gpartial, int pstride, double bytes, double flops)
{
    const ZSlot* zs = zbatch_slots();
    const int nz = zs ? zbatch_count() : 1;
    const int ps = std::max(pstride, J->ntiles[p]);
    struct {
        void* psi;
        void* lam;
        const void* ops;
        const double* mats;
        double* gpart;
        const void* zs;
        int op_first;
        int pstride;
    } args{psi, lam, ops + op_first, mats, gpartial, zs, op_first, ps};
    size_t asz = sizeof(args);
    void* cfg[] = {HIP_LAUNCH_PARAM_BUFFER_POINTER, &args, HIP_LAUNCH_PARAM_BUFFER_SIZE, &asz, HIP_LAUNCH_PARAM_END};
    ++g_launches_bwd;
    const int pi = prof_begin(YAO_KF_PASS_BWD);
    YAO_HIP(hipModuleLaunchKernel(J->fn[p], (unsigned)J->ntiles[p], (unsigned)J->nslots[p], (unsigned)nz, (unsigned)J->nthr[p], 1, 1, 0,
                                  stream(), nullptr, cfg));
    prof_end(pi, bytes * nz, flops * nz);
    return 0;
}

void jit_stats(long long* out)
{
    out[0] = g_compiled_programs.load();
    out[1] = g_compiled_passes.load();
    out[2] = g_failures.load();
    out[3] = g_launches_fwd.load();
    out[4] = g_launches_bwd.load();
}

void jit_free(JitPasses* J)
{
    if (!J) return;
    for (hipModule_t m : J->mod)
        if (m) (void)hipModuleUnload(m);
    delete J;
}

}  // namespace yao
