// Program kernels: evaluate a compiled site-local expression (see
// su3_program.cpp) at every site.  Most programs with matrix values run in
// the row form (k_program_rows, below); k_program takes the rest, one site
// per lane.  The operand fields
// the program reads are loaded into registers 0 .. nops-1 up front, so all
// of a lane's loads are in flight together; the instructions then run on
// registers, each a uniform branch on the opcode (matrix programs through
// an accumulator, below), and the result register is stored.
//
// A register holds a 3x3 complex matrix (NE = 9; a scalar uses entry 0).
// Programs without matrix values run in their own kernel, whose registers
// hold one complex value for each of the lane's S sites; programs whose
// every value is real (operands, intermediates and result, as in the
// real-valued composite example of Section 3, Listing 2) in a third, whose registers hold one real per site.  Register
// indices are uniform across the wave and are resolved by a chain of
// compare-and-copy branches, so the register file stays in VGPRs.
#include <type_traits>

#include "su3_device.h"
#include "su3_program.h"

namespace su3k {
namespace prog {

using su3i::ProgArgs;
using su3i::ProgInstr;

template <class T, int NE>
struct Reg {
    Cx<T> m[NE];
};

// End of a branch that wrote registers: an empty asm statement with an
// immediate unique to the branch, so that no two branches are merged into
// one copy through a selected address (which would move the register file
// to scratch memory).
template <int N>
__device__ __forceinline__ void branch_end()
{
    __asm__ volatile("" ::"n"(N));
}

struct NoReg {};

template <class T, int NE, int NR, int K>
using RegIf = typename std::conditional<(K < NR), Reg<T, NE>, NoReg>::type;

// The register file as separate members (never an indexable array).
template <class T, int NE, int NR>
struct RegFile {
    RegIf<T, NE, NR, 0> r0;
    RegIf<T, NE, NR, 1> r1;
    RegIf<T, NE, NR, 2> r2;
    RegIf<T, NE, NR, 3> r3;
    RegIf<T, NE, NR, 4> r4;
    RegIf<T, NE, NR, 5> r5;
    RegIf<T, NE, NR, 6> r6;
    RegIf<T, NE, NR, 7> r7;

    template <int K>
    __device__ __forceinline__ RegIf<T, NE, NR, K> &at()
    {
        if constexpr (K == 0) return r0;
        else if constexpr (K == 1) return r1;
        else if constexpr (K == 2) return r2;
        else if constexpr (K == 3) return r3;
        else if constexpr (K == 4) return r4;
        else if constexpr (K == 5) return r5;
        else if constexpr (K == 6) return r6;
        else return r7;
    }
};

template <class T, int NE, int NR, int K = 0>
__device__ __forceinline__ void get(RegFile<T, NE, NR> &R, int i, Reg<T, NE> &out)
{
    if constexpr (K < NR) {
        if (i == K) {
            out = R.template at<K>();
            branch_end<K>();
        } else {
            get<T, NE, NR, K + 1>(R, i, out);
        }
    }
}

template <class T, int NE, int NR, int K = 0>
__device__ __forceinline__ void put(RegFile<T, NE, NR> &R, int i, const Reg<T, NE> &v)
{
    if constexpr (K < NR) {
        if (i == K) {
            R.template at<K>() = v;
            branch_end<K + 16>();
        } else {
            put<T, NE, NR, K + 1>(R, i, v);
        }
    }
}

template <class T>
__device__ __forceinline__ Cx<T> cmul(Cx<T> a, Cx<T> b)
{
    return {fma_t(a.re, b.re, -(a.im * b.im)), fma_t(a.re, b.im, a.im * b.re)};
}

// Load a matrix operand of storage precision P into r (F32 arithmetic for
// F32 and the compressed form, whose third row is rebuilt).
template <int P, int NT>
__device__ __forceinline__ void load_matrix(const void *base, const su3i::Geom &g,
                                            uint32_t s, Reg<typename PrecT<P>::T, 9> &r)
{
    constexpr int E = PrecT<P>::E;
    RawVec<P, 1> raw[E];
    load_entries<P, 1, NT, true, 0, E>(static_cast<const typename PrecT<P>::R *>(base),
                                       site_offset(g, s), g.plane, 1, raw);
#pragma unroll
    for (int e = 0; e < E; ++e)
        r.m[e] = widen<P, 1>(raw[e], 0);
    if constexpr (P == su3i::C12)
        rebuild_row2(r.m);
}

template <class T, int NE, int NT>
__device__ __forceinline__ void load_operand(const ProgArgs &a, int k, uint32_t s,
                                             Reg<T, NE> &r)
{
    const void *base = a.op[k];
    switch (a.kind[k]) {
    case su3i::FK_MATRIX:
        if constexpr (NE == 9) {
            if constexpr (sizeof(T) == 8) {
                load_matrix<su3i::F64, NT>(base, a.g[k], s, r);
                branch_end<32>();
            } else {
                if (a.prec[k] == su3i::C12) {
                    load_matrix<su3i::C12, NT>(base, a.g[k], s, r);
                    branch_end<33>();
                } else {
                    load_matrix<su3i::F32, NT>(base, a.g[k], s, r);
                    branch_end<34>();
                }
            }
        }
        break;
    case su3i::FK_REAL:
        r.m[0] = {vload<NT & 1>(static_cast<const T *>(base) + s), T(0)};
        branch_end<35>();
        break;
    default: {  // complex scalar
        using V2 = typename VecOf<T, 2>::type;
        const V2 v = vload<NT & 1>(static_cast<const V2 *>(base) + s);
        r.m[0] = {v[0], v[1]};
        branch_end<36>();
        break;
    }
    }
}

// Matrix-form instructions work on an accumulator X: X holds r[a] when an
// instruction starts (it is copied in only when it holds another register)
// and r[d] when it ends (it is copied out every time, so the register file
// stays current).  A binary instruction reads r[b] in place through a
// branch per register, so the kernel keeps the file, X and a row of
// temporaries live instead of three matrix copies.

// X = X * B, one row at a time (row i of the product needs row i of X
// only); each entry is summed as in mat_mul.
template <class T>
__device__ __forceinline__ void mul_into(Reg<T, 9> &X, const Reg<T, 9> &B)
{
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        Cx<T> r[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            T re = X.m[3 * i].re * B.m[j].re;
            T im = X.m[3 * i].re * B.m[j].im;
            re = fma_t(-X.m[3 * i].im, B.m[j].im, re);
            im = fma_t(X.m[3 * i].im, B.m[j].re, im);
#pragma unroll
            for (int k = 1; k < 3; ++k) {
                re = fma_t(X.m[3 * i + k].re, B.m[3 * k + j].re, re);
                re = fma_t(-X.m[3 * i + k].im, B.m[3 * k + j].im, re);
                im = fma_t(X.m[3 * i + k].re, B.m[3 * k + j].im, im);
                im = fma_t(X.m[3 * i + k].im, B.m[3 * k + j].re, im);
            }
            r[j] = {re, im};
        }
#pragma unroll
        for (int j = 0; j < 3; ++j)
            X.m[3 * i + j] = r[j];
    }
}

// X = X (op) B for the binary opcodes OP_ADD_MM .. OP_SUB_MS.  Where a
// scalar X meets a matrix B, entry 0 of X is read by every entry of the
// result and is overwritten last.
template <class T>
__device__ __forceinline__ void binary(int op, Reg<T, 9> &X, const Reg<T, 9> &B)
{
    switch (op) {
    case su3i::OP_ADD_SS:
        X.m[0] = {X.m[0].re + B.m[0].re, X.m[0].im + B.m[0].im};
        break;
    case su3i::OP_SUB_SS:
        X.m[0] = {X.m[0].re - B.m[0].re, X.m[0].im - B.m[0].im};
        break;
    case su3i::OP_MUL_SS:
        X.m[0] = cmul(X.m[0], B.m[0]);
        break;
    case su3i::OP_ADD_MM:
#pragma unroll
        for (int e = 0; e < 9; ++e)
            X.m[e] = {X.m[e].re + B.m[e].re, X.m[e].im + B.m[e].im};
        break;
    case su3i::OP_SUB_MM:
#pragma unroll
        for (int e = 0; e < 9; ++e)
            X.m[e] = {X.m[e].re - B.m[e].re, X.m[e].im - B.m[e].im};
        break;
    case su3i::OP_MUL_MM:
        mul_into(X, B);
        break;
    case su3i::OP_MUL_SM:
#pragma unroll
        for (int e = 8; e >= 0; --e)
            X.m[e] = cmul(X.m[0], B.m[e]);
        break;
    case su3i::OP_MUL_MS:
#pragma unroll
        for (int e = 0; e < 9; ++e)
            X.m[e] = cmul(X.m[e], B.m[0]);
        break;
    case su3i::OP_ADD_SM:
#pragma unroll
        for (int e = 8; e >= 0; --e)
            X.m[e] = e % 4 == 0 ? Cx<T>{X.m[0].re + B.m[e].re, X.m[0].im + B.m[e].im} : B.m[e];
        break;
    case su3i::OP_ADD_MS:
#pragma unroll
        for (int e = 0; e < 9; e += 4)
            X.m[e] = {X.m[e].re + B.m[0].re, X.m[e].im + B.m[0].im};
        break;
    case su3i::OP_SUB_SM:
#pragma unroll
        for (int e = 8; e >= 0; --e)
            X.m[e] = e % 4 == 0 ? Cx<T>{X.m[0].re - B.m[e].re, X.m[0].im - B.m[e].im}
                                : Cx<T>{-B.m[e].re, -B.m[e].im};
        break;
    default:  // OP_SUB_MS
#pragma unroll
        for (int e = 0; e < 9; e += 4)
            X.m[e] = {X.m[e].re - B.m[0].re, X.m[e].im - B.m[0].im};
        break;
    }
}

// The binary instruction with r[i] as B, read where it lives.
template <class T, int NR, int K = 0>
__device__ __forceinline__ void binary_with(RegFile<T, 9, NR> &R, int i, int op, Reg<T, 9> &X)
{
    if constexpr (K < NR) {
        if (i == K) {
            binary<T>(op, X, R.template at<K>());
            branch_end<K + 48>();
        } else {
            binary_with<T, NR, K + 1>(R, i, op, X);
        }
    }
}

// X = op(X) for the other opcodes (OP_CONST ignores X and sets imm[a]).
template <class T>
__device__ __forceinline__ void unary(const ProgInstr in, const ProgArgs &a, Reg<T, 9> &X)
{
    switch (in.op) {
    case su3i::OP_CONST:
        X.m[0] = {T(a.imm[in.a][0]), T(a.imm[in.a][1])};
        break;
    case su3i::OP_NEG_S:
        X.m[0] = {-X.m[0].re, -X.m[0].im};
        break;
    case su3i::OP_CONJ_S:
        X.m[0] = {X.m[0].re, -X.m[0].im};
        break;
    case su3i::OP_REAL:
        X.m[0] = {X.m[0].re, T(0)};
        break;
    case su3i::OP_IMAG:
        X.m[0] = {X.m[0].im, T(0)};
        break;
    case su3i::OP_NEG_M:
#pragma unroll
        for (int e = 0; e < 9; ++e)
            X.m[e] = {-X.m[e].re, -X.m[e].im};
        break;
    case su3i::OP_CONJ_M:
#pragma unroll
        for (int e = 0; e < 9; ++e)
            X.m[e] = {X.m[e].re, -X.m[e].im};
        break;
    case su3i::OP_ADJ_M:
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            X.m[4 * i].im = -X.m[4 * i].im;
#pragma unroll
            for (int j = i + 1; j < 3; ++j) {
                const Cx<T> u = X.m[3 * i + j], v = X.m[3 * j + i];
                X.m[3 * i + j] = {v.re, -v.im};
                X.m[3 * j + i] = {u.re, -u.im};
            }
        }
        break;
    case su3i::OP_TRANS_M:
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = i + 1; j < 3; ++j) {
                const Cx<T> u = X.m[3 * i + j];
                X.m[3 * i + j] = X.m[3 * j + i];
                X.m[3 * j + i] = u;
            }
        break;
    case su3i::OP_TRACE:
        X.m[0] = {(X.m[0].re + X.m[4].re) + X.m[8].re, (X.m[0].im + X.m[4].im) + X.m[8].im};
        break;
    default:
        break;
    }
}

template <class T, int NE>
__device__ __forceinline__ void exec(const ProgInstr in, const ProgArgs &a,
                                     const Reg<T, NE> &A, const Reg<T, NE> &B,
                                     Reg<T, NE> &C)
{
    switch (in.op) {
    case su3i::OP_CONST:
        C.m[0] = {T(a.imm[in.a][0]), T(a.imm[in.a][1])};
        branch_end<96>();
        break;
    case su3i::OP_ADD_SS:
        C.m[0] = {A.m[0].re + B.m[0].re, A.m[0].im + B.m[0].im};
        branch_end<97>();
        break;
    case su3i::OP_SUB_SS:
        C.m[0] = {A.m[0].re - B.m[0].re, A.m[0].im - B.m[0].im};
        branch_end<98>();
        break;
    case su3i::OP_MUL_SS:
        C.m[0] = cmul(A.m[0], B.m[0]);
        branch_end<99>();
        break;
    case su3i::OP_NEG_S:
        C.m[0] = {-A.m[0].re, -A.m[0].im};
        branch_end<100>();
        break;
    case su3i::OP_CONJ_S:
        C.m[0] = {A.m[0].re, -A.m[0].im};
        branch_end<101>();
        break;
    case su3i::OP_REAL:
        C.m[0] = {A.m[0].re, T(0)};
        branch_end<102>();
        break;
    case su3i::OP_IMAG:
        C.m[0] = {A.m[0].im, T(0)};
        branch_end<103>();
        break;
    default:
        branch_end<104>();
        break;
    }
}

template <class T, int NE, int NR, int NT, int K = 0>
__device__ __forceinline__ void load_all(const ProgArgs &a, uint32_t s,
                                         RegFile<T, NE, NR> &R)
{
    if constexpr (K < NR) {
        if (K < a.nops) {
            if ((a.used >> K) & 1)
                load_operand<T, NE, NT>(a, K, s, R.template at<K>());
            load_all<T, NE, NR, NT, K + 1>(a, s, R);
        }
    }
}

template <class T, int NE, int NR, int NT>
__global__ __launch_bounds__(256) void k_program(ProgArgs a)
{
    extern __shared__ char occupancy_reserve[];
    const uint32_t group = a.xcd_remap ? (uint32_t)xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint32_t s = group * blockDim.x + threadIdx.x;
    if (s < (uint32_t)a.nsites) {
        RegFile<T, NE, NR> R;
        load_all<T, NE, NR, NT>(a, s, R);
        Reg<T, NE> Z;   // the accumulator
        int held = -1;  // the register Z is a copy of (the same in every lane)
        for (int pc = 0; pc < a.ninstr; ++pc) {
            const ProgInstr in = a.ins[pc];
            if (in.op != su3i::OP_CONST && in.a != held)
                get(R, in.a, Z);
            if (in.op >= su3i::OP_ADD_MM && in.op <= su3i::OP_SUB_MS)
                binary_with<T, NR>(R, in.b, in.op, Z);
            else
                unary<T>(in, a, Z);
            put(R, in.d, Z);
            held = in.d;
        }
        if (a.result != held)
            get(R, a.result, Z);
        switch (a.zkind) {
        case su3i::FK_MATRIX:
            if constexpr (NE == 9) {
                if constexpr (sizeof(T) == 8) {
                    RawVec<su3i::F64, 1> raw[9];
#pragma unroll
                    for (int e = 0; e < 9; ++e)
                        narrow<su3i::F64, 1>(raw[e], 0, Z.m[e]);
                    store_entries<su3i::F64, 1, NT, true, 0, 9>(
                        static_cast<double *>(a.z), site_offset(a.gz, s), a.gz.plane, 1, raw);
                } else if (a.zprec == su3i::C12) {
                    RawVec<su3i::C12, 1> raw[6];
#pragma unroll
                    for (int e = 0; e < 6; ++e)
                        narrow<su3i::C12, 1>(raw[e], 0, Z.m[e]);
                    store_entries<su3i::C12, 1, NT, true, 0, 6>(
                        static_cast<float *>(a.z), site_offset(a.gz, s), a.gz.plane, 1, raw);
                } else {
                    RawVec<su3i::F32, 1> raw[9];
#pragma unroll
                    for (int e = 0; e < 9; ++e)
                        narrow<su3i::F32, 1>(raw[e], 0, Z.m[e]);
                    store_entries<su3i::F32, 1, NT, true, 0, 9>(
                        static_cast<float *>(a.z), site_offset(a.gz, s), a.gz.plane, 1, raw);
                }
            }
            break;
        case su3i::FK_REAL:
            vstore<NT & 2>(static_cast<T *>(a.z) + s, Z.m[0].re);
            break;
        default: {
            using V2 = typename VecOf<T, 2>::type;
            V2 v;
            v[0] = Z.m[0].re;
            v[1] = Z.m[0].im;
            vstore<NT & 2>(static_cast<V2 *>(a.z) + s, v);
            break;
        }
        }
    }
    if (a.nsites < 0)
        occupancy_reserve[threadIdx.x] = 0;
}

// ------------------------------------------- matrix programs, row by row
//
// The row form (su3_program.h): three waves of a workgroup hold the three
// rows of every matrix value of 64 lanes' sites (S per lane: 16 bytes per
// entry and lane), wave r the row r.  Values live in LDS slots of 9 entries,
// so an instruction's operand is an address -- no selection of registers by
// chains of branches and copies, which cost the one-lane interpreter more
// than its arithmetic (force term FP64 32^4: 1130 VALU instructions a wave,
// some 250 of them arithmetic) -- and a lane needs registers for a few rows
// only: the waves a CU holds are set by the slots a program needs (9.1 KiB
// each), 24 for two slots, 12 for four, against 4 in double for the one-lane
// kernel.  What bounds it is the latency of LDS and memory those waves hide:
// a six-slot program holds the values no other wave reads in registers and
// so fits four slots.  Measured, one-lane kernel and here:
// (a*b+c*d)*(a*c+b*d)+(a-b)*(c-d) FP64 32^4 303 -> 219 us (755 MB), 8^4 18.6
// -> 9.1, FP32 48^4 560 -> 517; a*b-adj(b)*adj(a) FP64 48^4 494 -> 369 (6.2
// TB/s), FP32 16^4 7.1 -> 5.7; trace(a*b*adj(c)*adj(d)) FP64 48^4 660 -> 553.
// The last result is also in the accumulator Z.  A product reads its right
// operand's rows, a transposed operand its columns and a trace its diagonal
// from the slots the other waves wrote; the host sets the barriers that need
// (before a read of rows written since the last barrier, before a write of a
// slot read by other waves since then).  A scalar is computed by all three
// waves, each with a copy of its own in the slot.  Entries are summed as in
// the one-lane kernel: the same bits.
constexpr int kRowLanes = 64;  // lanes per row: a wave
// Vectors from one entry to the next: an odd count, so that whole AoS
// records (entries side by side) go into a slot without bank conflicts.
constexpr int kRowEntry = kRowLanes + 1;
constexpr int kRowSlot = 9 * kRowEntry;
static_assert(kRowSlot == su3i::kRowSlotVecs, "the host sizes LDS by it");

template <class T, int S>
struct RowVal {
    Cx<T> m[3][S];
};

// Forms of the kernel, or'ed.
enum RowForm {
    ROWF_HELD = 1,  // the code uses registers
    ROWF_AOS = 2,   // operands and result pass through LDS as whole records
};

template <class T, int S>
struct RowFrame {
    using V = typename VecOf<T, 2 * S>::type;
    V *own;  // entry (row, 0) of this lane's sites in slot 0
    V *all;  // entry (0, 0)
    int row;
    RowVal<T, S> Z, W0, W1;  // accumulator, registers
};

static_assert(su3i::kRowRegisters == 2, "held() and hold() name them");

template <bool HELD, class T, int S>
__device__ __forceinline__ RowVal<T, S> held(int src, const RowFrame<T, S> &f)
{
    if constexpr (!HELD)
        return f.Z;
    const bool z = src == su3i::ROW_ACC, w = src == su3i::ROW_ACC + 1;
    RowVal<T, S> x;
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const Cx<T> zv = f.Z.m[j][q], wv = f.W0.m[j][q], vv = f.W1.m[j][q];
            x.m[j][q] = {z ? zv.re : w ? wv.re : vv.re, z ? zv.im : w ? wv.im : vv.im};
        }
    return x;
}

template <class T, int S>
__device__ __forceinline__ void hold(int d, const RowVal<T, S> &x, RowFrame<T, S> &f)
{
    const bool w = d == su3i::ROW_ACC + 1;
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const Cx<T> v = x.m[j][q], w0 = f.W0.m[j][q], w1 = f.W1.m[j][q];
            f.W0.m[j][q] = {w ? v.re : w0.re, w ? v.im : w0.im};
            f.W1.m[j][q] = {w ? w1.re : v.re, w ? w1.im : v.im};
        }
}

template <class T, int S>
__device__ __forceinline__ void unpack(const typename VecOf<T, 2 * S>::type &v, Cx<T> (&c)[S])
{
#pragma unroll
    for (int q = 0; q < S; ++q)
        c[q] = {v[2 * q], v[2 * q + 1]};
}

template <class T, int S>
__device__ __forceinline__ typename VecOf<T, 2 * S>::type pack(const Cx<T> (&c)[S])
{
    typename VecOf<T, 2 * S>::type v;
#pragma unroll
    for (int q = 0; q < S; ++q) {
        v[2 * q] = c[q].re;
        v[2 * q + 1] = c[q].im;
    }
    return v;
}

template <int N, class T, int S>
__device__ __forceinline__ void apply_mode(int mode, RowVal<T, S> &x)
{
    if (mode & su3i::ROW_CONJ) {
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int q = 0; q < S; ++q)
                x.m[j][q].im = -x.m[j][q].im;
    }
    if (mode & su3i::ROW_NEG) {
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int q = 0; q < S; ++q)
                x.m[j][q] = {-x.m[j][q].re, -x.m[j][q].im};
    }
}

// This wave's row of a matrix source.
template <bool HELD, class T, int S>
__device__ __forceinline__ RowVal<T, S> row_of(int src, int mode, const RowFrame<T, S> &f)
{
    RowVal<T, S> x;
    if (src & su3i::ROW_ACC) {
        x = held<HELD>(src, f);
    } else if (mode & su3i::ROW_TRANS) {
        const auto *p = f.all + src * kRowSlot + f.row * kRowEntry;
#pragma unroll
        for (int j = 0; j < 3; ++j)
            unpack<T, S>(p[3 * j * kRowEntry], x.m[j]);
    } else {
        const auto *p = f.own + src * kRowSlot;
#pragma unroll
        for (int j = 0; j < 3; ++j)
            unpack<T, S>(p[j * kRowEntry], x.m[j]);
    }
    apply_mode<3>(mode, x);
    return x;
}

// A scalar source, in x.m[0] (this wave's copy: entry (row, 0)).
template <bool HELD, class T, int S>
__device__ __forceinline__ RowVal<T, S> scalar_of(int src, int mode, const su3i::RowArgs &a,
                                                  const RowFrame<T, S> &f)
{
    RowVal<T, S> x;
    if (src & su3i::ROW_ACC) {
        x = held<HELD>(src, f);
    } else if (src & su3i::ROW_IMM) {
        const int k = src & 7;
#pragma unroll
        for (int q = 0; q < S; ++q)
            x.m[0][q] = {T(a.imm[k][0]), T(a.imm[k][1])};
    } else {
        unpack<T, S>(f.own[src * kRowSlot], x.m[0]);
    }
    apply_mode<1>(mode, x);
    return x;
}

// Row of A * B, entry (k, j) of B at b[k * SK + j * SJ]; each entry is
// summed over k as in mat_mul.
template <int SK, int SJ, class T, int S>
__device__ __forceinline__ void row_product(const RowVal<T, S> &A,
                                            const typename VecOf<T, 2 * S>::type *b, bool conj,
                                            RowVal<T, S> &z)
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        RowVal<T, S> e;
#pragma unroll
        for (int j = 0; j < 3; ++j)
            unpack<T, S>(b[k * SK + j * SJ], e.m[j]);
        if (conj)
            apply_mode<3>(su3i::ROW_CONJ, e);
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const Cx<T> x = A.m[k][q], y = e.m[j][q];
                Cx<T> &c = z.m[j][q];
                if (k == 0) {
                    c.re = x.re * y.re;
                    c.im = x.re * y.im;
                } else {
                    c.re = fma_t(x.re, y.re, c.re);
                }
                c.re = fma_t(-x.im, y.im, c.re);
                if (k != 0)
                    c.im = fma_t(x.re, y.im, c.im);
                c.im = fma_t(x.im, y.re, c.im);
            }
    }
}

// Row f.row of operand k (or the scalar) of the S sites from s0 into its
// slot's registers.  Loads are whole vectors: fields are padded to whole
// lane-blocks of a multiple of S.
template <int P, int S, int NT>
__device__ __forceinline__ void load_row(const void *base, const su3i::Geom &g, uint32_t s0,
                                         int row, RowVal<typename PrecT<P>::T, S> &r)
{
    using R = typename PrecT<P>::R;
    const R *p = static_cast<const R *>(base);
    const uint32_t off = site_offset(g, s0);
    if (P == su3i::C12 && row == 2) {  // rebuilt from rows 0 and 1
        RawVec<P, S> raw[6];
        load_entries<P, S, NT, true, 0, 6>(p, off, g.plane, S, raw);
#pragma unroll
        for (int q = 0; q < S; ++q) {
            Cx<typename PrecT<P>::T> m[9];
#pragma unroll
            for (int e = 0; e < 6; ++e)
                m[e] = widen<P, S>(raw[e], q);
            rebuild_row2(m);
#pragma unroll
            for (int j = 0; j < 3; ++j)
                r.m[j][q] = m[6 + j];
        }
    } else {
        RawVec<P, S> raw[3];
        load_entries<P, S, NT, true, 0, 3>(p, off + 3 * row * g.plane, g.plane, S, raw);
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int q = 0; q < S; ++q)
                r.m[j][q] = widen<P, S>(raw[j], q);
    }
}

template <class T, int S, int NT>
__device__ __forceinline__ void load_row_operand(const su3i::RowArgs &a, int k, uint32_t s0,
                                                 int row, RowVal<T, S> &r)
{
    const void *base = a.op[k];
    if (a.kind[k] == su3i::FK_MATRIX) {
        if constexpr (sizeof(T) == 8)
            load_row<su3i::F64, S, NT>(base, a.g[k], s0, row, r);
        else if (a.prec[k] == su3i::C12)
            load_row<su3i::C12, S, NT>(base, a.g[k], s0, row, r);
        else
            load_row<su3i::F32, S, NT>(base, a.g[k], s0, row, r);
    } else if (a.kind[k] == su3i::FK_REAL) {
        const T *p = static_cast<const T *>(base) + s0;
        if constexpr (S == 1) {
            r.m[0][0] = {vload<NT & 1>(p), T(0)};
        } else {
            using V = typename VecOf<T, S>::type;
            const V v = vload<NT & 1>(reinterpret_cast<const V *>(p));
#pragma unroll
            for (int q = 0; q < S; ++q)
                r.m[0][q] = {v[q], T(0)};
        }
    } else {
        using V = typename VecOf<T, 2 * S>::type;
        unpack<T, S>(vload<NT & 1>(reinterpret_cast<const V *>(static_cast<const T *>(base) +
                                                               2 * s0)),
                     r.m[0]);
    }
}

// The operands into their slots, four at a time (their loads in flight
// together).
template <int FORM, class T, int S, int NT>
__device__ __forceinline__ void load_slots(const su3i::RowArgs &a, uint32_t s0, bool inside,
                                           RowFrame<T, S> &f)
{
    for (int k0 = 0; k0 < a.nops; k0 += 4) {
        RowVal<T, S> v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (inside && k0 + i < a.nops && ((a.used >> (k0 + i)) & 1))
                load_row_operand<T, S, NT>(a, k0 + i, s0, f.row, v[i]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (inside && k0 + i < a.nops && ((a.used >> (k0 + i)) & 1)) {
                if ((FORM & ROWF_HELD) && (a.slot[k0 + i] & su3i::ROW_ACC)) {
                    hold(a.slot[k0 + i], v[i], f);
                    continue;
                }
                auto *p = f.own + a.slot[k0 + i] * kRowSlot;
                p[0] = pack<T, S>(v[i].m[0]);
                if (a.kind[k0 + i] == su3i::FK_MATRIX) {
                    p[kRowEntry] = pack<T, S>(v[i].m[1]);
                    p[2 * kRowEntry] = pack<T, S>(v[i].m[2]);
                }
            }
    }
}

// AoS operands: the workgroup's 64 sites are 576 consecutive entries of each
// matrix, read as they lie and put in place by entry and site; the rest (two-
// row matrices, scalars) as above.
template <class T, int NT>
__device__ __forceinline__ void load_slots_aos(const su3i::RowArgs &a, uint32_t first,
                                               bool inside, int lane, const RowFrame<T, 1> &f)
{
    using V = typename VecOf<T, 2>::type;
    constexpr int kVecs = 9 * kRowLanes, kThreads = 3 * kRowLanes;
    V *const slots = f.all - lane;
    const uint32_t nvec = 9u * (uint32_t)a.nsites;
    const uint32_t t = (uint32_t)f.row * kRowLanes + lane;
    for (int k = 0; k < a.nops; ++k) {
        if (!((a.used >> k) & 1))
            continue;
        if (a.kind[k] != su3i::FK_MATRIX || a.prec[k] == su3i::C12) {
            if (inside) {
                RowVal<T, 1> r;
                load_row_operand<T, 1, NT>(a, k, first + lane, f.row, r);
                V *p = f.own + a.slot[k] * kRowSlot;
                p[0] = pack<T, 1>(r.m[0]);
                if (a.kind[k] == su3i::FK_MATRIX) {
                    p[kRowEntry] = pack<T, 1>(r.m[1]);
                    p[2 * kRowEntry] = pack<T, 1>(r.m[2]);
                }
            }
            continue;
        }
        const V *g = static_cast<const V *>(a.op[k]);
        V v[kVecs / kThreads];
#pragma unroll
        for (int i = 0; i < kVecs / kThreads; ++i) {
            const uint32_t at = 9u * first + t + i * kThreads;
            if (at < nvec)
                v[i] = vload<NT & 1>(g + at);
        }
#pragma unroll
        for (int i = 0; i < kVecs / kThreads; ++i) {
            const uint32_t e = t + i * kThreads;
            if (9u * first + e < nvec)
                slots[a.slot[k] * kRowSlot + (e % 9) * kRowEntry + e / 9] = v[i];
        }
    }
    __syncthreads();  // rows were written by every wave
}

// Row `row` of a matrix result in storage precision P (cnt of the S sites).
template <int P, int S, int NT>
__device__ __forceinline__ void store_row(const su3i::RowArgs &a, uint32_t s0, int row, int cnt,
                                          const RowVal<typename PrecT<P>::T, S> &Z)
{
    using R = typename PrecT<P>::R;
    RawVec<P, S> raw[3];
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int q = 0; q < S; ++q)
            narrow<P, S>(raw[j], q, Z.m[j][q]);
    const uint32_t off = site_offset(a.gz, s0) + 3 * row * a.gz.plane;
    if (cnt >= S)
        store_entries<P, S, NT, true, 0, 3>(static_cast<R *>(a.z), off, a.gz.plane, S, raw);
    else
        store_entries<P, S, NT, false, 0, 3>(static_cast<R *>(a.z), off, a.gz.plane, cnt, raw);
}

template <class T, int S, int NT, int FORM>
__global__ __launch_bounds__(3 * kRowLanes) void k_program_rows(su3i::RowArgs a)
{
    extern __shared__ char occupancy_reserve[];
    constexpr bool HELD = FORM & ROWF_HELD, AOS = FORM & ROWF_AOS;
    using V = typename RowFrame<T, S>::V;
    V *const slots = reinterpret_cast<V *>(occupancy_reserve);
    const int row = __builtin_amdgcn_readfirstlane(threadIdx.x / kRowLanes);
    const int lane = threadIdx.x % kRowLanes;
    RowFrame<T, S> f;
    f.own = slots + 3 * row * kRowEntry + lane;
    f.all = slots + lane;
    f.row = row;
    const uint32_t group = a.xcd_remap ? (uint32_t)xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint32_t first = group * (kRowLanes * S);  // the workgroup's first site
    const uint32_t s0 = first + lane * S;
    const bool inside = s0 < (uint32_t)a.nsites;  // lanes past the end only take part
    if constexpr (AOS)
        load_slots_aos<T, NT>(a, first, inside, lane, f);
    else
        load_slots<FORM, T, S, NT>(a, s0, inside, f);
    RowVal<T, S> &Z = f.Z;
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int q = 0; q < S; ++q)
            Z.m[j][q] = {T(0), T(0)};
    su3i::RowInstr next = a.ins[0];
    for (int pc = 0; pc < a.ninstr; ++pc) {
        const su3i::RowInstr in = next;
        next = a.ins[pc + 1 < a.ninstr ? pc + 1 : pc];
        if (in.flags & su3i::ROW_SYNC_READ)
            __syncthreads();
        switch (in.op) {
        case su3i::ROW_MUL_M: {
            const RowVal<T, S> A = row_of<HELD>(in.a, in.am, f);
            const V *b = f.all + in.b * kRowSlot;
            const bool conj = in.bm & su3i::ROW_CONJ;
            if (in.bm & su3i::ROW_TRANS)
                row_product<kRowEntry, 3 * kRowEntry>(A, b, conj, Z);
            else
                row_product<3 * kRowEntry, kRowEntry>(A, b, conj, Z);
            break;
        }
        case su3i::ROW_ADD_M: {
            const RowVal<T, S> A = row_of<HELD>(in.a, in.am, f);
            const RowVal<T, S> B = row_of<HELD>(in.b, in.bm, f);
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int q = 0; q < S; ++q)
                    Z.m[j][q] = {A.m[j][q].re + B.m[j][q].re, A.m[j][q].im + B.m[j][q].im};
            break;
        }
        case su3i::ROW_MOV_M: Z = row_of<HELD>(in.a, in.am, f); break;
        case su3i::ROW_MUL_SM: {
            const RowVal<T, S> A = scalar_of<HELD>(in.a, in.am, a, f);
            const RowVal<T, S> B = row_of<HELD>(in.b, in.bm, f);
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int q = 0; q < S; ++q)
                    Z.m[j][q] = cmul(A.m[0][q], B.m[j][q]);
            break;
        }
        case su3i::ROW_MUL_MS: {
            const RowVal<T, S> A = row_of<HELD>(in.a, in.am, f);
            const RowVal<T, S> B = scalar_of<HELD>(in.b, in.bm, a, f);
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int q = 0; q < S; ++q)
                    Z.m[j][q] = cmul(A.m[j][q], B.m[0][q]);
            break;
        }
        case su3i::ROW_ADD_MS: {
            const RowVal<T, S> B = scalar_of<HELD>(in.b, in.bm, a, f);
            Z = row_of<HELD>(in.a, in.am, f);
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (j == row)
#pragma unroll
                    for (int q = 0; q < S; ++q)
                        Z.m[j][q] = {Z.m[j][q].re + B.m[0][q].re,
                                     Z.m[j][q].im + B.m[0][q].im};
            break;
        }
        case su3i::ROW_TRACE: {
            const V *p = f.all + in.a * kRowSlot;
            RowVal<T, S> d;
#pragma unroll
            for (int j = 0; j < 3; ++j)
                unpack<T, S>(p[4 * j * kRowEntry], d.m[j]);
            apply_mode<3>(in.am, d);
#pragma unroll
            for (int q = 0; q < S; ++q)
                Z.m[0][q] = {(d.m[0][q].re + d.m[1][q].re) + d.m[2][q].re,
                             (d.m[0][q].im + d.m[1][q].im) + d.m[2][q].im};
            break;
        }
        default: {  // scalars
            const RowVal<T, S> A = scalar_of<HELD>(in.a, in.am, a, f);
            if (in.op == su3i::ROW_ADD_S || in.op == su3i::ROW_MUL_S) {
                const RowVal<T, S> B = scalar_of<HELD>(in.b, in.bm, a, f);
#pragma unroll
                for (int q = 0; q < S; ++q)
                    Z.m[0][q] = in.op == su3i::ROW_MUL_S
                                    ? cmul(A.m[0][q], B.m[0][q])
                                    : Cx<T>{A.m[0][q].re + B.m[0][q].re,
                                            A.m[0][q].im + B.m[0][q].im};
            } else {
#pragma unroll
                for (int q = 0; q < S; ++q)
                    Z.m[0][q] = in.op == su3i::ROW_REAL   ? Cx<T>{A.m[0][q].re, T(0)}
                                : in.op == su3i::ROW_IMAG ? Cx<T>{A.m[0][q].im, T(0)}
                                                          : A.m[0][q];
            }
            break;
        }
        }
        if (in.d & su3i::ROW_ACC) {
            if constexpr (HELD)
                if (in.d != su3i::ROW_NONE)
                    hold(in.d, Z, f);
        } else {
            if (in.flags & su3i::ROW_SYNC_WRITE)
                __syncthreads();
            V *p = f.own + in.d * kRowSlot;
#pragma unroll
            for (int j = 0; j < 3; ++j)
                p[j * kRowEntry] = pack<T, S>(Z.m[j]);
        }
    }
    if constexpr (AOS) {
        if (a.zkind == su3i::FK_MATRIX && a.zprec != su3i::C12) {
            // the rows back through a slot, out as whole vectors
            constexpr int kThreads = 3 * kRowLanes;
            const uint32_t nvec = 9u * (uint32_t)a.nsites, t = threadIdx.x;
            __syncthreads();  // every wave is done with slot 0
#pragma unroll
            for (int j = 0; j < 3; ++j)
                f.own[j * kRowEntry] = pack<T, 1>(Z.m[j]);
            __syncthreads();
            V *g = static_cast<V *>(a.z);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const uint32_t e = t + i * kThreads;
                if (9u * first + e < nvec)
                    vstore<NT & 2>(g + 9u * first + e, slots[(e % 9) * kRowEntry + e / 9]);
            }
            return;
        }
    }
    if (!inside)
        return;
    const int left = a.nsites - (int)s0, cnt = left < S ? left : S;
    if (a.zkind == su3i::FK_MATRIX) {
        if constexpr (sizeof(T) == 8) {
            store_row<su3i::F64, S, NT>(a, s0, row, cnt, Z);
        } else if (a.zprec == su3i::C12) {
            if (row < 2)
                store_row<su3i::C12, S, NT>(a, s0, row, cnt, Z);
        } else {
            store_row<su3i::F32, S, NT>(a, s0, row, cnt, Z);
        }
    } else if (row == 0) {
        T *z = static_cast<T *>(a.z);
        if (a.zkind == su3i::FK_REAL) {
#pragma unroll
            for (int q = 0; q < S; ++q)
                if (q < cnt)
                    vstore<NT & 2>(z + s0 + q, Z.m[0][q].re);
        } else {
            using V2 = typename VecOf<T, 2>::type;
#pragma unroll
            for (int q = 0; q < S; ++q)
                if (q < cnt) {
                    V2 v;
                    v[0] = Z.m[0][q].re;
                    v[1] = Z.m[0][q].im;
                    vstore<NT & 2>(reinterpret_cast<V2 *>(z) + s0 + q, v);
                }
        }
    }
}

// Scalar-only programs: each lane evaluates S sites (one complex value per
// site in each register), so a site costs 1/S of the instruction dispatch.
// A lane's sites are S / W vectors of W, W the sites of 16 bytes of a complex
// field (1 in double, 2 in single): vector q of lane l in the lane group
// g = gid / 64 is vector (S / W g + q) * 64 + l of the field, so each access
// of a wave is 1 KiB of consecutive bytes (512 of a real field).  Bound by
// memory: with 4 (double) or 8 (single) sites side by side in a lane, 16
// bytes 64 apart, nontemporal loads fetched every line four times (a*conj(b)+a
// FP32 48^4, 127 MB: 172 us, now 26.6; FP64, 255 MB: 161, now 46), and the
// smallest lattices waited for eight sites' copies (FP32 8^4 8.9, now 5.2).
template <class T>
constexpr int kScalarVec = 8 / sizeof(T);

template <class T, int S>
struct SReg {
    Cx<T> v[S];
};

// Vectors v0 + 64 q; vectors past the end read as 0.
template <class T, int S, int NT>
__device__ __forceinline__ void load_scalars(const ProgArgs &a, int k, uint32_t v0, uint32_t n,
                                             SReg<T, S> &r)
{
    constexpr int W = kScalarVec<T>;
    const bool real = a.kind[k] == su3i::FK_REAL;
#pragma unroll
    for (int q = 0; q < S / W; ++q) {
        const uint32_t s0 = (v0 + 64u * q) * W;
        if (s0 + W <= n) {
            if (real) {
                const T *p = static_cast<const T *>(a.op[k]) + s0;
                if constexpr (W == 1) {
                    r.v[q] = {vload<NT & 1>(p), T(0)};
                } else {
                    using V = typename VecOf<T, W>::type;
                    const V w = vload<NT & 1>(reinterpret_cast<const V *>(p));
#pragma unroll
                    for (int j = 0; j < W; ++j)
                        r.v[q * W + j] = {w[j], T(0)};
                }
                branch_end<40>();
            } else {
                using V = typename VecOf<T, 2 * W>::type;
                const V w = vload<NT & 1>(
                    reinterpret_cast<const V *>(static_cast<const T *>(a.op[k]) + 2 * s0));
#pragma unroll
                for (int j = 0; j < W; ++j)
                    r.v[q * W + j] = {w[2 * j], w[2 * j + 1]};
                branch_end<41>();
            }
        } else {
            const T *p = static_cast<const T *>(a.op[k]);
#pragma unroll
            for (int j = 0; j < W; ++j) {
                r.v[q * W + j] = {T(0), T(0)};
                if (s0 + j < n) {
                    if (real)
                        r.v[q * W + j].re = p[s0 + j];
                    else
                        r.v[q * W + j] = {p[2 * (s0 + j)], p[2 * (s0 + j) + 1]};
                }
            }
        }
    }
}

template <class T, int S, int NT>
__device__ __forceinline__ void store_scalars(const ProgArgs &a, uint32_t v0, uint32_t n,
                                              const SReg<T, S> &Z)
{
    constexpr int W = kScalarVec<T>;
    T *z = static_cast<T *>(a.z);
#pragma unroll
    for (int q = 0; q < S / W; ++q) {
        const uint32_t s0 = (v0 + 64u * q) * W;
        if (a.zkind == su3i::FK_REAL) {
            if (W > 1 && s0 + W <= n) {
                using V = typename VecOf<T, W>::type;
                V w;
#pragma unroll
                for (int j = 0; j < W; ++j)
                    w[j] = Z.v[q * W + j].re;
                vstore<NT & 2>(reinterpret_cast<V *>(z + s0), w);
            } else {
#pragma unroll
                for (int j = 0; j < W; ++j)
                    if (s0 + j < n)
                        vstore<NT & 2>(z + s0 + j, Z.v[q * W + j].re);
            }
        } else if (s0 + W <= n) {
            using V = typename VecOf<T, 2 * W>::type;
            V w;
#pragma unroll
            for (int j = 0; j < W; ++j) {
                w[2 * j] = Z.v[q * W + j].re;
                w[2 * j + 1] = Z.v[q * W + j].im;
            }
            vstore<NT & 2>(reinterpret_cast<V *>(z + 2 * s0), w);
        } else {
#pragma unroll
            for (int j = 0; j < W; ++j)
                if (s0 + j < n) {
                    z[2 * (s0 + j)] = Z.v[q * W + j].re;
                    z[2 * (s0 + j) + 1] = Z.v[q * W + j].im;
                }
        }
    }
}

template <class T, int S>
__device__ __forceinline__ void exec_scalars(const ProgInstr in, const ProgArgs &a,
                                             const SReg<T, S> &A, const SReg<T, S> &B,
                                             SReg<T, S> &C)
{
#pragma unroll
    for (int j = 0; j < S; ++j) {
        Reg<T, 1> x, y, z;
        x.m[0] = A.v[j];
        y.m[0] = B.v[j];
        exec<T, 1>(in, a, x, y, z);
        C.v[j] = z.m[0];
    }
}

template <class T, int S, int NR, int K = 0>
__device__ __forceinline__ void sget(RegFile<T, S, NR> &R, int i, SReg<T, S> &out)
{
    if constexpr (K < NR) {
        if (i == K) {
            const Reg<T, S> &r = R.template at<K>();
#pragma unroll
            for (int j = 0; j < S; ++j)
                out.v[j] = r.m[j];
            branch_end<K + 48>();
        } else {
            sget<T, S, NR, K + 1>(R, i, out);
        }
    }
}

template <class T, int S, int NR, int K = 0>
__device__ __forceinline__ void sput(RegFile<T, S, NR> &R, int i, const SReg<T, S> &v)
{
    if constexpr (K < NR) {
        if (i == K) {
            Reg<T, S> &r = R.template at<K>();
#pragma unroll
            for (int j = 0; j < S; ++j)
                r.m[j] = v.v[j];
            branch_end<K + 56>();
        } else {
            sput<T, S, NR, K + 1>(R, i, v);
        }
    }
}

template <class T, int S, int NR, int NT, int K = 0>
__device__ __forceinline__ void sload_all(const ProgArgs &a, uint32_t v0, uint32_t n,
                                          RegFile<T, S, NR> &R)
{
    if constexpr (K < NR) {
        if (K < a.nops) {
            if ((a.used >> K) & 1) {
                SReg<T, S> t;
                load_scalars<T, S, NT>(a, K, v0, n, t);
                sput<T, S, NR>(R, K, t);
            }
            sload_all<T, S, NR, NT, K + 1>(a, v0, n, R);
        }
    }
}

// Registers here hold S sites' values (RegFile entries reused as S-wide).
template <class T, int S, int NR, int NT>
__global__ __launch_bounds__(256) void k_program_scalar(ProgArgs a)
{
    extern __shared__ char occupancy_reserve[];
    constexpr int W = kScalarVec<T>;
    const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t v0 = (gid >> 6) * (64u * (S / W)) + (gid & 63u);
    const uint32_t n = (uint32_t)a.nsites;
    if (a.nsites > 0 && v0 * W < n) {
        RegFile<T, S, NR> R;
        sload_all<T, S, NR, NT>(a, v0, n, R);
        for (int pc = 0; pc < a.ninstr; ++pc) {
            const ProgInstr in = a.ins[pc];
            SReg<T, S> A, B, C;
            sget(R, in.a, A);
            sget(R, in.b, B);
            exec_scalars<T, S>(in, a, A, B, C);
            sput(R, in.d, C);
        }
        SReg<T, S> Z;
        sget(R, a.result, Z);
        store_scalars<T, S, NT>(a, v0, n, Z);
    }
    if (a.nsites < 0)
        occupancy_reserve[threadIdx.x] = 0;
}

// ------------------------------------------------ real-valued programs
//
// Every operand, intermediate and the result are real fields (one value
// per site).  A lane holds S = 2 W sites in each register, W = values per
// 16-byte vector: vector q (0, 1) of lane l in the lane group g = gid / 64
// is vector (2 g + q) * 64 + l of the field, so each load and store
// instruction of a wave moves 1 KiB of consecutive bytes.  Block sizes
// are multiples of 64, so the lane groups are the hardware waves.

template <class T, int S>
struct RVal {
    T v[S];
};

template <class T, int S, int NR, int K>
using RValIf = typename std::conditional<(K < NR), RVal<T, S>, NoReg>::type;

template <class T, int S, int NR>
struct RealFile {
    RValIf<T, S, NR, 0> r0;
    RValIf<T, S, NR, 1> r1;
    RValIf<T, S, NR, 2> r2;
    RValIf<T, S, NR, 3> r3;
    RValIf<T, S, NR, 4> r4;
    RValIf<T, S, NR, 5> r5;
    RValIf<T, S, NR, 6> r6;
    RValIf<T, S, NR, 7> r7;

    template <int K>
    __device__ __forceinline__ RValIf<T, S, NR, K> &at()
    {
        if constexpr (K == 0) return r0;
        else if constexpr (K == 1) return r1;
        else if constexpr (K == 2) return r2;
        else if constexpr (K == 3) return r3;
        else if constexpr (K == 4) return r4;
        else if constexpr (K == 5) return r5;
        else if constexpr (K == 6) return r6;
        else return r7;
    }
};

template <class T, int S, int NR, int K = 0>
__device__ __forceinline__ void rget(RealFile<T, S, NR> &R, int i, RVal<T, S> &out)
{
    if constexpr (K < NR) {
        if (i == K) {
            out = R.template at<K>();
            branch_end<K + 112>();
        } else {
            rget<T, S, NR, K + 1>(R, i, out);
        }
    }
}

template <class T, int S, int NR, int K = 0>
__device__ __forceinline__ void rput(RealFile<T, S, NR> &R, int i, const RVal<T, S> &v)
{
    if constexpr (K < NR) {
        if (i == K) {
            R.template at<K>() = v;
            branch_end<K + 120>();
        } else {
            rput<T, S, NR, K + 1>(R, i, v);
        }
    }
}

// The lane's values of a real field p of n sites; v0 = the lane's first
// vector.  Sites past n read as zero.
template <class T, int S, int NT>
__device__ __forceinline__ void rload(const T *p, uint32_t v0, uint32_t n, RVal<T, S> &r)
{
    constexpr int W = 16 / sizeof(T);
    using V = typename VecOf<T, W>::type;
#pragma unroll
    for (int q = 0; q < S / W; ++q) {
        const uint32_t vi = v0 + 64u * q, s = vi * W;
        if (s + W <= n) {
            const V w = vload<NT & 1>(reinterpret_cast<const V *>(p) + vi);
#pragma unroll
            for (int j = 0; j < W; ++j)
                r.v[q * W + j] = w[j];
        } else {
#pragma unroll
            for (int j = 0; j < W; ++j)
                r.v[q * W + j] = s + j < n ? p[s + j] : T(0);
        }
    }
}

template <class T, int S, int NT>
__device__ __forceinline__ void rstore(T *p, uint32_t v0, uint32_t n, const RVal<T, S> &r)
{
    constexpr int W = 16 / sizeof(T);
    using V = typename VecOf<T, W>::type;
#pragma unroll
    for (int q = 0; q < S / W; ++q) {
        const uint32_t vi = v0 + 64u * q, s = vi * W;
        if (s + W <= n) {
            V w;
#pragma unroll
            for (int j = 0; j < W; ++j)
                w[j] = r.v[q * W + j];
            vstore<NT & 2>(reinterpret_cast<V *>(p) + vi, w);
        } else {
#pragma unroll
            for (int j = 0; j < W; ++j)
                if (s + j < n)
                    p[s + j] = r.v[q * W + j];
        }
    }
}

// One instruction on S sites: one branch on the opcode for all of them.
// Real values take only the real-closed opcodes (constants are real, the
// conjugate and the real part are the identity, the imaginary part is
// zero).
template <class T, int S>
__device__ __forceinline__ void exec_real(const ProgInstr in, const ProgArgs &a,
                                          const RVal<T, S> &A, const RVal<T, S> &B,
                                          RVal<T, S> &C)
{
    switch (in.op) {
    case su3i::OP_CONST: {
        const T c = T(a.imm[in.a][0]);
#pragma unroll
        for (int j = 0; j < S; ++j)
            C.v[j] = c;
        branch_end<128>();
        break;
    }
    case su3i::OP_ADD_SS:
#pragma unroll
        for (int j = 0; j < S; ++j)
            C.v[j] = A.v[j] + B.v[j];
        branch_end<129>();
        break;
    case su3i::OP_SUB_SS:
#pragma unroll
        for (int j = 0; j < S; ++j)
            C.v[j] = A.v[j] - B.v[j];
        branch_end<130>();
        break;
    case su3i::OP_MUL_SS:
#pragma unroll
        for (int j = 0; j < S; ++j)
            C.v[j] = A.v[j] * B.v[j];
        branch_end<131>();
        break;
    case su3i::OP_NEG_S:
#pragma unroll
        for (int j = 0; j < S; ++j)
            C.v[j] = -A.v[j];
        branch_end<132>();
        break;
    case su3i::OP_IMAG:
#pragma unroll
        for (int j = 0; j < S; ++j)
            C.v[j] = T(0);
        branch_end<133>();
        break;
    default:  // OP_CONJ_S, OP_REAL
        C = A;
        branch_end<134>();
        break;
    }
}

template <class T, int S, int NR, int NT, int K = 0>
__device__ __forceinline__ void rload_all(const ProgArgs &a, uint32_t v0, uint32_t n,
                                          RealFile<T, S, NR> &R)
{
    if constexpr (K < NR) {
        if (K < a.nops) {
            if ((a.used >> K) & 1) {
                RVal<T, S> t;
                rload<T, S, NT>(static_cast<const T *>(a.op[K]), v0, n, t);
                rput<T, S, NR>(R, K, t);
            }
            rload_all<T, S, NR, NT, K + 1>(a, v0, n, R);
        }
    }
}

template <class T, int S, int NR, int NT>
__global__ __launch_bounds__(256) void k_program_real(ProgArgs a)
{
    extern __shared__ char occupancy_reserve[];
    constexpr int W = 16 / sizeof(T);
    const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t v0 = (gid >> 6) * (64u * (S / W)) + (gid & 63u);
    const uint32_t n = (uint32_t)a.nsites;
    if (a.nsites > 0 && v0 * W < n) {
        RealFile<T, S, NR> R;
        rload_all<T, S, NR, NT>(a, v0, n, R);
        for (int pc = 0; pc < a.ninstr; ++pc) {
            const ProgInstr in = a.ins[pc];
            RVal<T, S> A, B, C;
            rget(R, in.a, A);
            rget(R, in.b, B);
            exec_real<T, S>(in, a, A, B, C);
            rput(R, in.d, C);
        }
        RVal<T, S> Z;
        rget(R, a.result, Z);
        rstore<T, S, NT>(static_cast<T *>(a.z), v0, n, Z);
    }
    if (a.nsites < 0)
        occupancy_reserve[threadIdx.x] = 0;
}

template <class T, int NE, int NR>
static hipError_t go(int nt, int block, int grid, size_t shm, const ProgArgs &a,
                     hipStream_t st)
{
    if ((nt & 3) == 3)
        hipLaunchKernelGGL((k_program<T, NE, NR, 3>), dim3(grid), dim3(block), shm, st, a);
    else if ((nt & 3) == 2)
        hipLaunchKernelGGL((k_program<T, NE, NR, 2>), dim3(grid), dim3(block), shm, st, a);
    else
        hipLaunchKernelGGL((k_program<T, NE, NR, 0>), dim3(grid), dim3(block), shm, st, a);
    return hipGetLastError();
}

template <class T, int S, int FORM>
static hipError_t go_rows(int nt, size_t shm, const su3i::RowArgs &a, hipStream_t st)
{
    const int per = kRowLanes * S;
    const dim3 grid((unsigned)(((int64_t)a.nsites + per - 1) / per)), block(3 * kRowLanes);
    const size_t need = (size_t)a.nslots * kRowSlot * S * 2 * sizeof(T);
    if (shm < need)
        shm = need;
    auto *k = (nt & 3) == 3   ? k_program_rows<T, S, 3, FORM>
              : (nt & 3) == 2 ? k_program_rows<T, S, 2, FORM>
                              : k_program_rows<T, S, 0, FORM>;
    if (shm > 64 * 1024) {
        // beyond the default dynamic LDS of a workgroup (eight slots take
        // 75 KB)
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)shm);
        if (e != hipSuccess)
            return e;
    }
    hipLaunchKernelGGL(k, grid, block, shm, st, a);
    return hipGetLastError();
}

template <class T, int S>
static hipError_t pick_rows(int nt, size_t shm, const su3i::RowArgs &a, hipStream_t st)
{
    if constexpr (S == 1) {
        if (a.aos)
            return a.held ? hipErrorInvalidValue : go_rows<T, 1, ROWF_AOS>(nt, shm, a, st);
    }
    return a.held ? go_rows<T, S, ROWF_HELD>(nt, shm, a, st) : go_rows<T, S, 0>(nt, shm, a, st);
}

// Sites per lane of real-valued programs: 32 bytes of each operand (two
// 16-byte accesses); of scalar-only ones 32 bytes of each complex operand.
template <class T>
constexpr int kRealSites = 32 / sizeof(T);
template <class T>
constexpr int kScalarSites = 16 / sizeof(T);

template <class T, int NR>
static hipError_t go_scalar(int nt, int block, int grid, size_t shm,
                            const ProgArgs &a, hipStream_t st)
{
    constexpr int S = kScalarSites<T>;
    if ((nt & 3) == 3)
        hipLaunchKernelGGL((k_program_scalar<T, S, NR, 3>), dim3(grid), dim3(block), shm, st, a);
    else if ((nt & 3) == 2)
        hipLaunchKernelGGL((k_program_scalar<T, S, NR, 2>), dim3(grid), dim3(block), shm, st, a);
    else
        hipLaunchKernelGGL((k_program_scalar<T, S, NR, 0>), dim3(grid), dim3(block), shm, st, a);
    return hipGetLastError();
}

template <class T, int NR>
static hipError_t go_real(int nt, int block, int grid, size_t shm,
                          const ProgArgs &a, hipStream_t st)
{
    constexpr int S = kRealSites<T>;
    if ((nt & 3) == 3)
        hipLaunchKernelGGL((k_program_real<T, S, NR, 3>), dim3(grid), dim3(block), shm, st, a);
    else if ((nt & 3) == 2)
        hipLaunchKernelGGL((k_program_real<T, S, NR, 2>), dim3(grid), dim3(block), shm, st, a);
    else
        hipLaunchKernelGGL((k_program_real<T, S, NR, 0>), dim3(grid), dim3(block), shm, st, a);
    return hipGetLastError();
}

template <class T>
static hipError_t go_t(int form, int nregs, int nt, int block, int grid,
                       size_t shm, const ProgArgs &a, hipStream_t st)
{
    if (form == su3i::PF_REAL)
        return nregs <= 4 ? go_real<T, 4>(nt, block, grid, shm, a, st)
                          : go_real<T, 8>(nt, block, grid, shm, a, st);
    if (form == su3i::PF_SCALAR)
        return nregs <= 4 ? go_scalar<T, 4>(nt, block, grid, shm, a, st)
                          : go_scalar<T, 8>(nt, block, grid, shm, a, st);
    // waves per SIMD the register file allows (double / single): 2 / 5
    // for two registers, 1 / 3 for four, 1 / 2 for eight (in double the
    // eight matrices fill the VGPRs and AGPRs of one wave)
    if (nregs <= 2)
        return go<T, 9, 2>(nt, block, grid, shm, a, st);
    if (nregs <= 4)
        return go<T, 9, 4>(nt, block, grid, shm, a, st);
    return go<T, 9, 8>(nt, block, grid, shm, a, st);
}

}  // namespace prog
}  // namespace su3k

namespace su3i {

int program_sites_per_lane(int arith, int form)
{
    if (form == PF_MATRIX)
        return 1;
    if (form == PF_REAL)
        return arith == F64 ? su3k::prog::kRealSites<double> : su3k::prog::kRealSites<float>;
    return arith == F64 ? su3k::prog::kScalarSites<double>
                        : su3k::prog::kScalarSites<float>;
}

hipError_t launch_program(int arith, int form, int nregs, int nt,
                          int block, int grid, size_t shm, const ProgArgs &a,
                          hipStream_t st)
{
    using namespace su3k::prog;
    if (block > 256 || block % 64 || nregs < 1 || nregs > kProgMaxRegs ||
        form < PF_MATRIX || form > PF_REAL)
        return hipErrorInvalidValue;
    if (arith == F64)
        return go_t<double>(form, nregs, nt, block, grid, shm, a, st);
    if (arith == F32)
        return go_t<float>(form, nregs, nt, block, grid, shm, a, st);
    return hipErrorInvalidValue;
}

hipError_t launch_program_rows(int arith, int sites_per_lane, int nt, size_t shm,
                               const RowArgs &a, hipStream_t st)
{
    using namespace su3k::prog;
    if (a.nsites < 1 || a.ninstr < 1 || a.ninstr > kProgMaxInstr || a.nslots < 1 ||
        a.nslots > kRowMaxSlots)
        return hipErrorInvalidValue;
    if (arith == F64 && sites_per_lane == 1)
        return pick_rows<double, 1>(nt, shm, a, st);
    if (arith == F32 && sites_per_lane == 1)
        return pick_rows<float, 1>(nt, shm, a, st);
    if (arith == F32 && sites_per_lane == 2 && !a.aos)
        return pick_rows<float, 2>(nt, shm, a, st);
    return hipErrorInvalidValue;
}

}  // namespace su3i
