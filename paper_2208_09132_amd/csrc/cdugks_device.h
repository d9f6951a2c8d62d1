// Device-side building blocks of the CDUGKS kernels (included by every
// kernel translation unit): storage access, primitives, the face-sum and
// update kernel bodies, and the per-face / per-cell closures.  The data
// layout and the structure of a step are described in cdugks_kernels.hip.
#pragma once

#include "cdugks_internal.h"

#include <math.h>

#include <type_traits>

namespace cdg {

__device__ __forceinline__ int map_coord(int x, int n, int bc) {
    if (bc == 0) {
        int r = x % n;
        return r < 0 ? r + n : r;
    }
    return x < 0 ? 0 : (x >= n ? n - 1 : x);
}

// Reciprocal from the hardware estimate (relative error below 1e-7) refined
// by one Newton-Raphson step, which squares the error to about 2e-15.  Used
// where the operand is a nonzero finite sum.
__device__ __forceinline__ double rcp_nr(double s) {
    const double r = __builtin_amdgcn_rcp(s);
    return fma(r, fma(-s, r, 1.0), r);
}

// Van Leer limiter (eq. VanLeer) at half scale: H(a, b) = ab/(a + b) when
// ab > 0, else 0, which is half the harmonic-mean form 2ab/(a+b) =
// (sgn a + sgn b)|a||b|/(|a|+|b|): zero at extrema and for a flat side.  The
// kernels carry every limited slope at half scale (and slopes of slopes at a
// quarter), folding the factors into the Courant numbers; all the scalings
// are powers of two, so the values are those of the full-scale form exactly
// (except where a product is subnormal, as in the far velocity tails of the
// FP32 form).
// When ab > 0 the sum a + b is nonzero, so the reciprocal is safe; otherwise
// its value is discarded by the select.
__device__ __forceinline__ double half_van_leer(double a, double b) {
    double p = a * b;
    double v = p * rcp_nr(a + b);
    return p > 0.0 ? v : 0.0;
}

// FP32 form for the FP32-storage stencil: the hardware reciprocal alone
// (within 1 ulp), so the limited slope is within about 2 ulp of the rounded
// quotient, below the rounding of the FP32 values it is built from and
// stored as.
__device__ __forceinline__ float half_van_leer(float a, float b) {
    float p = a * b;
    float v = p * __builtin_amdgcn_rcpf(a + b);
    return p > 0.0f ? v : 0.0f;
}

template <typename ST>
__device__ __forceinline__ double ld(const void* base, long long idx) {
    return (double)reinterpret_cast<const ST*>(base)[idx];
}
template <typename ST>
__device__ __forceinline__ void st(void* base, long long idx, double v) {
    reinterpret_cast<ST*>(base)[idx] = (ST)v;
}

// Streaming store for data the writing kernel never reads again (face values,
// the new distributions): marked non-temporal so it does not push the halo
// lines that neighbouring workgroups still need out of L2.
template <typename ST>
__device__ __forceinline__ void st_stream(void* base, long long idx, double v) {
    __builtin_nontemporal_store((ST)v, reinterpret_cast<ST*>(base) + idx);
}

// A 32-bit offset that the compiler takes as new at this point.  An address
// formed from a uniform row and a 32-bit offset costs no VALU instruction, but
// only where the widening to 64 bits stands beside the access: of an offset
// that is constant over a loop it would be moved out, leaving a 64-bit sum per
// access inside.
__device__ __forceinline__ void keep_offset(unsigned& b) {
#ifdef __HIP_DEVICE_COMPILE__
    asm("" : "+v"(b));
#else
    (void)b;
#endif
}
// the element `b` bytes into a row (a uniform base)
template <typename E>
__device__ __forceinline__ E at_byte(const E* row, unsigned b) {
    return *(const E*)((const char*)row + b);
}
// Face-value stores, NF values fstride apart.  A streaming (non-temporal) store
// of part of a 64-byte sector is written out as it is, and the memory reads,
// merges and writes the sector again, while an ordinary one meets the
// neighbouring tile's part in L2.  So rows of the face grid that do not start
// on whole sectors (P.fv_stream = 0) take ordinary stores: streaming against
// ordinary, face sums: 191^2 x 21^2 FP64 441 / 273 us, 310^2 x 18^2 FP32 551 /
// 377 us, 41^3 x 10^3 FP32 2.81 / 1.38 ms.  On whole sectors streaming wins in
// FP64, as the update then finds g and b in L2 (256^2 x 28^2, both phases: 1348
// / 1385 us); in FP32, whose 16-wide tile rows are one sector, only over 4096
// velocities and more (256^2 cells x 28^2, 64^2, 80^2, 129^2: 896 / 885, 4830 /
// 4860, 7430 / 7760, 19300 / 20160 us), which fv_streams leaves out below that.
enum { FV_STREAM = 0, FV_ORDINARY = 1, FV_EITHER = 2 };
// What a face-sum kernel takes unless told otherwise: 1-D tiles are rows of
// whole lines; a test per store (EITHER) costs the 2-D kernels 2%, the 3-D ones
// nothing.
template <int D>
constexpr int fv_store_mode() { return D == 1 ? FV_STREAM : (D == 2 ? FV_ORDINARY : FV_EITHER); }
// row: the value's row (uniform), b: its byte offset there, 32 bits as in the
// update: with 64-bit sums per load and store the z-march, bound by VALU issue,
// took 4 to 5 registers more and 32^3 FP32 cells 1009 us for the face sums
// instead of 987, 37 x 29 x 23 cells 743 instead of 695 (FP64 storage 1396
// instead of 1379)
template <typename ST, int NF, int MODE>
__device__ __forceinline__ void st_faces_row(const Problem& P, ST* row, unsigned b, long long fstride,
                                             const ST (&v)[NF]) {
    unsigned bk[NF];
#pragma unroll
    for (int k = 0; k < NF; ++k) {
        bk[k] = b;
        keep_offset(bk[k]);
    }
    auto at = [&](int k) __attribute__((always_inline)) { return (ST*)((char*)(row + k * fstride) + bk[k]); };
    if (MODE == FV_STREAM || (MODE == FV_EITHER && P.fv_stream)) {  // uniform
        if constexpr (MODE == FV_EITHER) asm volatile("; streaming");
#pragma unroll
        for (int k = 0; k < NF; ++k) __builtin_nontemporal_store(v[k], at(k));
        if constexpr (MODE == FV_EITHER) asm volatile("; streaming");
    } else {
#pragma unroll
        for (int k = 0; k < NF; ++k) *at(k) = v[k];
    }
}
template <typename ST, int NF, int MODE>
__device__ __forceinline__ void st_faces(const Problem& P, long long o, long long fstride, const ST (&v)[NF]) {
    ST* const p = (ST*)P.FV + o;
    if (MODE == FV_STREAM || (MODE == FV_EITHER && P.fv_stream)) {  // uniform
        // an (empty) difference between the branches, before and after: alike
        // but for the streaming mark they would be merged into one without it
        if constexpr (MODE == FV_EITHER) asm volatile("; streaming");
#pragma unroll
        for (int k = 0; k < NF; ++k) __builtin_nontemporal_store(v[k], p + k * fstride);
        if constexpr (MODE == FV_EITHER) asm volatile("; streaming");
    } else {
#pragma unroll
        for (int k = 0; k < NF; ++k) p[k * fstride] = v[k];
    }
}

__device__ __forceinline__ void raise_error(int* err) { *err = 1; }

// ---------------------------------------------------------------------------
// storage forms of the distributions g, b (and of the 3-D quarter-step fields)
// ---------------------------------------------------------------------------
// double, float: every velocity row [N] in that precision.
// Bf16Tail: the FP32 form, except that the rows of the far velocity tails
// (fixed at set-up) hold BF16.  P.rows[i] is the byte offset of row i inside
// each state array, with bit 0 set for a BF16 row.  The stencil arithmetic
// and the stored face values are FP32 as in the FP32 form.  Values are
// rounded to FP32 and then, in a BF16 row, to BF16 (round to nearest even).
struct Bf16Tail {};

template <typename ST>
struct StoreT {
    using C = ST;  // stencil arithmetic and stored face values
    using R = ST;  // a loaded state value, as held in registers until used
    static constexpr bool MIXED = false;
};
template <>
struct StoreT<Bf16Tail> {
    using C = float;
    using R = unsigned;  // raw bits: the FP32 word, or the BF16 half zero-extended
    static constexpr bool MIXED = true;
};

// row word of velocity i (uniform: a scalar load)
__device__ __forceinline__ long long row_word(const Problem& P, int i) {
    return ((const __attribute__((address_space(4))) long long*)(const void*)P.rows)[i];
}

// state value at (velocity i, cell c), raw until state_value converts it
template <typename ST>
__device__ __forceinline__ typename StoreT<ST>::R state_load(const Problem& P, const void* base, int i,
                                                            long long c) {
    if constexpr (StoreT<ST>::MIXED) {
        const long long o = row_word(P, i);
        const char* row = (const char*)base + (o & ~1LL);
        if (o & 1) return (unsigned)((const unsigned short*)row)[c];
        return ((const unsigned*)row)[c];
    } else {
        return ((const ST*)base)[(long long)i * P.pitch + c];
    }
}
template <typename ST>
__device__ __forceinline__ double state_value(const Problem& P, int i, typename StoreT<ST>::R r) {
    if constexpr (StoreT<ST>::MIXED) {
        return (double)__uint_as_float((row_word(P, i) & 1) ? r << 16 : r);
    } else {
        return (double)r;
    }
}
template <typename ST>
__device__ __forceinline__ double state_ld(const Problem& P, const void* base, int i, long long c) {
    return state_value<ST>(P, i, state_load<ST>(P, base, i, c));
}
template <typename ST, bool STREAM>
__device__ __forceinline__ void state_st(const Problem& P, void* base, int i, long long c, double v) {
    if constexpr (StoreT<ST>::MIXED) {
        const long long o = row_word(P, i);
        char* row = (char*)base + (o & ~1LL);
        const float f = (float)v;
        if (o & 1) {
            const unsigned short h = __builtin_bit_cast(unsigned short, (__bf16)f);
            if constexpr (STREAM) __builtin_nontemporal_store(h, (unsigned short*)row + c);
            else ((unsigned short*)row)[c] = h;
        } else {
            if constexpr (STREAM) __builtin_nontemporal_store(f, (float*)row + c);
            else ((float*)row)[c] = f;
        }
    } else {
        if constexpr (STREAM) st_stream<ST>(base, (long long)i * P.pitch + c, v);
        else st<ST>(base, (long long)i * P.pitch + c, v);
    }
}

// The fields of velocity i at NS source cells of one thread, raw until
// slot_value.  The BF16-tail form has two ways to read a row whose kind is
// uniform per velocity:
//  WORDS: one 32-bit load per slot whatever the row's kind (element c of a
//    BF16 row is a half of word c/2, which slot_value takes out), so no branch
//    on the row kind stands between these loads and the values that use them
//    (at a branch's join the compiler waits for every load in flight).  The
//    word of a BF16 row's last element reaches past the row's 2N bytes only
//    for an odd N, into the padding that rounds the row to 256 bytes.  For
//    loops over velocities.
//  !WORDS: 16-bit loads under a branch on the row kind (the value in the low
//    half, as for an even cell), for a velocity fixed over the loop.
template <typename ST, int NS, bool WORDS = true>
__device__ __forceinline__ void load_slots(const Problem& P, const void* sg, const void* sb, int i,
                                           const long long (&src)[NS], typename StoreT<ST>::R (&og)[NS],
                                           typename StoreT<ST>::R (&ob)[NS]) {
    if constexpr (StoreT<ST>::MIXED && WORDS) {
        const long long o = row_word(P, i);
        const int h = (int)(o & 1);
        const unsigned* rg = (const unsigned*)((const char*)sg + (o & ~1LL));
        const unsigned* rb = (const unsigned*)((const char*)sb + (o & ~1LL));
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            const long long w = src[k] >> h;
            og[k] = rg[w];
            ob[k] = rb[w];
        }
    } else if constexpr (StoreT<ST>::MIXED) {
        const long long o = row_word(P, i);
        const char* rg = (const char*)sg + (o & ~1LL);
        const char* rb = (const char*)sb + (o & ~1LL);
        if (o & 1) {
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                og[k] = ((const unsigned short*)rg)[src[k]];
                ob[k] = ((const unsigned short*)rb)[src[k]];
            }
        } else {
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                og[k] = ((const unsigned*)rg)[src[k]];
                ob[k] = ((const unsigned*)rb)[src[k]];
            }
        }
    } else {
        // the row's base address is uniform (scalar) and the cell offsets
        // are loop-invariant, so each load is a scalar base plus a fixed
        // vector offset
        const ST* const rg = (const ST*)sg + (long long)i * P.pitch;
        const ST* const rb = (const ST*)sb + (long long)i * P.pitch;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            og[k] = rg[src[k]];
            ob[k] = rb[src[k]];
        }
    }
}
// value of a raw slot of cell c: in a BF16 row (half, uniform) a word loaded
// by WORDS holds cells c and c ^ 1, the odd cell in the upper half; a 16-bit
// load is passed as an even cell
template <typename ST>
__device__ __forceinline__ double slot_value(typename StoreT<ST>::R r, bool half, long long c) {
    if constexpr (StoreT<ST>::MIXED) {
        const unsigned bits = half ? ((c & 1) ? (r & 0xFFFF0000u) : (r << 16)) : r;
        return (double)__uint_as_float(bits);
    } else {
        return (double)r;
    }
}

// Access within one velocity row of the update kernel, whose element kind is
// known at compile time: double or float rows, or the BF16 rows of the
// BF16-tail form (Bf16Row).  `off` is the row's byte offset in the array.
// Stores are non-temporal (the kernel never reads them back); round() gives
// the value as it will be stored.
struct Bf16Row {};
template <typename E>
struct RowIO {
    using Raw = E;  // a loaded element, as held until used
    static constexpr int BYTES = sizeof(E);
    // element c of the row, or (raw_at, st_at) the one b bytes into it
    __device__ static Raw raw(const void* base, long long off, long long c) {
        return ((const E*)((const char*)base + off))[c];
    }
    __device__ static Raw raw_at(const void* base, long long off, unsigned b) {
        return at_byte((const E*)((const char*)base + off), b);
    }
    __device__ static double val(Raw r) { return (double)r; }
    __device__ static void st(void* base, long long off, long long c, double v) {
        __builtin_nontemporal_store((E)v, (E*)((char*)base + off) + c);
    }
    __device__ static void st_at(void* base, long long off, unsigned b, double v) {
        __builtin_nontemporal_store((E)v, (E*)((char*)base + off + b));
    }
    __device__ static double round(double v) { return (double)(E)v; }
};
template <>
struct RowIO<Bf16Row> {
    using Raw = __bf16;
    static constexpr int BYTES = 2;
    __device__ static Raw raw(const void* base, long long off, long long c) {
        return ((const __bf16*)((const char*)base + off))[c];
    }
    __device__ static Raw raw_at(const void* base, long long off, unsigned b) {
        return at_byte((const __bf16*)((const char*)base + off), b);
    }
    __device__ static double val(Raw r) { return (double)(float)r; }
    __device__ static void st(void* base, long long off, long long c, double v) {
        st_at(base, off + 2 * c, 0, v);
    }
    __device__ static void st_at(void* base, long long off, unsigned b, double v) {
        const unsigned short h = __builtin_bit_cast(unsigned short, (__bf16)(float)v);
        __builtin_nontemporal_store(h, (unsigned short*)((char*)base + off + b));
    }
    __device__ static double round(double v) { return (double)(float)(__bf16)(float)v; }
};

// ---------------------------------------------------------------------------
// primitives shared by the per-cell and per-face closures (Sec. 2)
// ---------------------------------------------------------------------------
struct Prim {
    double rho, u[3], RT, inv_tau_g;
    bool bad;
};

__device__ __forceinline__ Prim primitives(const Problem& P, int D, const double* Wv) {
    Prim q;
    q.rho = Wv[0];
    double u2 = 0.0;
    for (int d = 0; d < 3; ++d) {
        q.u[d] = d < D ? Wv[1 + d] / q.rho : 0.0;
        u2 += q.u[d] * q.u[d];
    }
    double E = Wv[D + 1] / q.rho;
    double T = (P.gamma - 1.0) / P.R * (E - 0.5 * u2);
    q.RT = P.R * T;
    if (P.relax == 0) {
        double mu = P.mu_ref * pow(T / P.T_ref, P.omega);
        q.inv_tau_g = q.rho * q.RT / mu;
    } else {
        q.inv_tau_g = P.tau_inv;
    }
    q.bad = !(q.rho > 0.0) || !(T > 0.0) || !isfinite(q.rho) || !isfinite(T) ||
            !isfinite(q.u[0]) || !isfinite(q.u[1]) || !isfinite(q.u[2]) || !isfinite(q.inv_tau_g);
    return q;
}

__device__ __forceinline__ double maxwell_prefactor(int D, double rho, double RT) {
    double two_pi_rt = 2.0 * M_PI * RT;
    double f = D == 1 ? 1.0 / sqrt(two_pi_rt)
                      : (D == 2 ? 1.0 / two_pi_rt : 1.0 / (two_pi_rt * sqrt(two_pi_rt)));
    return rho * f;
}

struct CellCoef {
    double A, inv2RT, cRT2, beta, betab, eta, hu2, u[3];
};

__device__ __forceinline__ CellCoef cell_coefs(const Problem& P, int D, const Prim& q) {
    CellCoef k;
    k.A = maxwell_prefactor(D, q.rho, q.RT);
    k.inv2RT = 0.5 / q.RT;
    k.cRT2 = 0.5 * P.c_int * q.RT;
    k.beta = 0.25 * P.dt * q.inv_tau_g;
    k.betab = k.beta * P.Pr;
    k.eta = k.beta * (P.Pr - 1.0);
    k.hu2 = 0.5 * (q.u[0] * q.u[0] + q.u[1] * q.u[1] + q.u[2] * q.u[2]);
#pragma unroll
    for (int d = 0; d < 3; ++d) k.u[d] = q.u[d];
    return k;
}

__device__ __forceinline__ void store_coef(double* Pc, long long N, long long c, const CellCoef& k) {
    Pc[PC_A * N + c] = k.A;
    Pc[PC_INV2RT * N + c] = k.inv2RT;
    Pc[PC_CRT2 * N + c] = k.cRT2;
    Pc[PC_BETA * N + c] = k.beta;
    Pc[PC_BETAB * N + c] = k.betab;
    Pc[PC_ETA * N + c] = k.eta;
    Pc[PC_HU2 * N + c] = k.hu2;
#pragma unroll
    for (int d = 0; d < 3; ++d) Pc[(PC_U0 + d) * N + c] = k.u[d];
}

// ---------------------------------------------------------------------------
// tile kernels
// ---------------------------------------------------------------------------
// XCD-aware order: consecutive workgroup ids are spread over the 8 XCDs, so
// give each XCD a contiguous block of the (tile, slice) space; neighbouring
// tiles then share halo lines in that XCD's L2.
__device__ __forceinline__ int xcd_remap(int lin, int total) {
    int per = total / 8;
    if (lin >= per * 8) return lin;
    return (lin % 8) * per + lin / 8;
}

// Box geometry of the staged halo for a face-sum tile: the q box covers tile
// offsets [-3, T+1], the limited-difference box [-2, T].  (The left face of
// cell c along d needs the upwind cell c-d or c, its slopes at the upwind
// cell +-1 along d, and those need q one further out.)
template <int D, int TID>
struct Geo {
    static constexpr TileExt T = tile_shape(D, TID);
    static constexpr int TX = T.x, TY = T.y, TZ = T.z;
    static constexpr int NT = TX * TY * TZ;  // threads of a workgroup, one per cell
    static constexpr int QX = TX + 5;
    static constexpr int QY = D >= 2 ? TY + 5 : 1;
    static constexpr int QZ = D >= 3 ? TZ + 5 : 1;
    static constexpr int AX = TX + 3;
    static constexpr int AY = D >= 2 ? TY + 3 : 1;
    static constexpr int AZ = D >= 3 ? TZ + 3 : 1;
    static constexpr int NQ = QX * QY * QZ;
    static constexpr int NA = AX * AY * AZ;
    static constexpr int NRA = (NA + NT - 1) / NT;   // slope points per thread
    static constexpr bool CACHE_COEF = (NQ - NT + NT - 1) / NT + 1 <= 2;
    // offsets of tile coordinate 0 inside the boxes, and box strides
    static constexpr int OQX = 3, OQY = D >= 2 ? 3 : 0, OQZ = D >= 3 ? 3 : 0;
    static constexpr int OAX = 2, OAY = D >= 2 ? 2 : 0, OAZ = D >= 3 ? 2 : 0;
    __device__ static constexpr int SQ(int e) { return e == 0 ? 1 : (e == 1 ? QX : QX * QY); }
    __device__ static constexpr int SA(int e) { return e == 0 ? 1 : (e == 1 ? AX : AX * AY); }
    __device__ static int qidx(int x, int y, int z) { return (x + OQX) + QX * ((y + OQY) + QY * (z + OQZ)); }
    __device__ static int aidx(int x, int y, int z) { return (x + OAX) + AX * ((y + OAY) + AY * (z + OAZ)); }
};

__device__ __forceinline__ CellCoef load_coef(const double* Pc, long long N, long long c) {
    CellCoef k;
    k.A = Pc[PC_A * N + c];
    k.inv2RT = Pc[PC_INV2RT * N + c];
    k.cRT2 = Pc[PC_CRT2 * N + c];
    k.beta = Pc[PC_BETA * N + c];
    k.betab = Pc[PC_BETAB * N + c];
    k.eta = Pc[PC_ETA * N + c];
    k.hu2 = Pc[PC_HU2 * N + c];
    k.u[0] = Pc[PC_U0 * N + c];
    k.u[1] = Pc[(PC_U0 + 1) * N + c];
    k.u[2] = Pc[(PC_U0 + 2) * N + c];
    return k;
}

struct Vel {
    double xi[3], w, hx2, lam2[3], ax;
};

// The velocity table is read-only for the whole launch: reading it through the
// constant address space makes the per-velocity loads scalar (SMEM), so they
// neither occupy vector-memory slots nor delay waits on the field loads.
typedef const __attribute__((address_space(4))) double* const_dptr;

__device__ __forceinline__ const_dptr vel_ptr(const double* vel, int i) {
    return (const_dptr)(const void*)(vel + (long long)i * NVEL);
}

__device__ __forceinline__ Vel load_vel(const double* vel, int i) {
    const_dptr v = vel_ptr(vel, i);
    Vel r;
    r.xi[0] = v[0]; r.xi[1] = v[1]; r.xi[2] = v[2];
    r.w = v[VE_W]; r.hx2 = v[VE_HX2]; r.ax = v[VE_AX];
    r.lam2[0] = v[VE_LAM0]; r.lam2[1] = v[VE_LAM0 + 1]; r.lam2[2] = v[VE_LAM0 + 2];
    return r;
}

// Z and the quarter-step fields at one (cell, velocity), given g_eq:
// phi_bar_plus = phi + (h/2)(phi_eq - phi)/tau + (h/2) S (eq. phibarplus),
// S_b = Z (g - g_eq)/tau_bg + ... .  ACC adds the external acceleration's
// terms of the sources (eqs. gsource, bsource) with the velocity derivative
// taken on the equilibrium: S_g = a.(xi - u)/(R T) g_eq and, in S_b,
// a.xi (g - g_eq) + a.(xi - u)/(R T) b_eq; (h/2)/(R T) = (dt/2)/(2 R T).
template <int D, bool ACC = false>
__device__ __forceinline__ void quarter_step_eq(const CellCoef& k, const Vel& v, double geq, double g, double b,
                                                double& qg, double& qb, const Problem* P = nullptr) {
    double xu = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) xu += v.xi[d] * k.u[d];
    double beq = (v.hx2 + k.cRT2) * geq;
    double Z = xu - k.hu2;
    qg = g + k.beta * (geq - g);
    qb = b + k.betab * (beq - b) + k.eta * Z * (g - geq);
    if constexpr (ACC) {
        double au = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) au += P->accel[d] * k.u[d];
        const double c = 0.5 * P->dt * k.inv2RT * (v.ax - au);
        qg += c * geq;
        qb += 0.25 * P->dt * v.ax * (g - geq) + c * beq;
    }
}

// Value of phi_bar at a face centre at t_{n+1/2} from the upwind cell u,
// side s = +1 when the face is u's right face, -1 when its left face:
//   v = q(u) + s a_d/2 - sum_e lambda_e (a_e + s b_de/2),
// a_e = VL of one-sided differences of q along e (slope times dx_e) and
// b_de = VL of differences of a_e along d (slope of the slope times dx_d dx_e).
// Arguments at the scales the kernels carry: ha = a/2 at u (haU) and at
// u - d (haL), u + d (haR); lam2 = 2 lambda.  Then
//   v = q(u) + s ha_d - sum_e lam2_e (ha_e + s hb_de),  hb_de = b_de/4 = H(ha differences).
template <int D, typename CT>
__device__ __forceinline__ CT face_value_at(CT qU, const CT* haU, const CT* haL, const CT* haR, int d, CT s,
                                            const Vel& v) {
    CT val = qU + s * haU[d];
#pragma unroll
    for (int e = 0; e < D; ++e) {
        CT hb = half_van_leer(haU[e] - haL[e], haR[e] - haU[e]);
        val -= CT(v.lam2[e]) * (haU[e] + s * hb);
    }
    return val;
}

// The single-slope option: the upwind cell's own slopes carried to the foot,
// v = q(u) + s ha_d - sum_e lam2_e ha_e (no slopes of slopes).
template <int D, typename CT>
__device__ __forceinline__ CT face_value_single(CT qU, const CT* haU, int d, CT s, const Vel& v) {
    CT val = qU + s * haU[d];
#pragma unroll
    for (int e = 0; e < D; ++e) val -= CT(v.lam2[e]) * haU[e];
    return val;
}

// Face coefficients used to invert eq. phibar at a face.  The inversion
// g = ig gbar + bg g_eq with bg = 1 - ig is evaluated as g_eq + ig (gbar -
// g_eq) (likewise b with ib), so bg and bb need no registers.
template <int D>
struct FaceCoef {
    double A, inv2RT, cRT2, ig, ib, eb, hu2, u[D];
    __device__ void load(const double* F, long long NE) {
        A = F[PF_A * NE];
        inv2RT = F[PF_INV2RT * NE];
        cRT2 = F[PF_CRT2 * NE];
        ig = F[PF_IG * NE];
        ib = F[PF_IB * NE];
        eb = F[PF_EB * NE];
        hu2 = F[PF_HU2 * NE];
#pragma unroll
        for (int e = 0; e < D; ++e) u[e] = F[(PF_U0 + e) * NE];
    }
    // Z = xi.u - |u|^2/2 at the face
    __device__ __forceinline__ double z(const Vel& v) const {
        double xu = 0.0;
#pragma unroll
        for (int e = 0; e < D; ++e) xu += v.xi[e] * u[e];
        return xu - hu2;
    }
    // phi at the face from phi_bar (eq. phibar inverted): g first, then b with
    // the S_b source at the face evaluated with the face g and Z = z(v).
    __device__ __forceinline__ void invert_z(const Vel& v, double geq, double Z, double vg, double vb, double& gF,
                                             double& bF) const {
        double beq = (v.hx2 + cRT2) * geq;
        gF = geq + ig * (vg - geq);
        bF = beq + ib * (vb - beq) + eb * Z * (gF - geq);
    }
    // The same with an external acceleration a: the face's (h/2) S terms
    // (eqs. gsource, bsource, velocity derivative on the equilibrium), with
    // au = a.u_f and c2 = (dt/2)/(2 R T_f) prepared once per face.
    double au, c2;
    __device__ void prepare_accel(const double* a, double dt) {
        au = 0.0;
#pragma unroll
        for (int e = 0; e < D; ++e) au += a[e] * u[e];
        c2 = 0.5 * dt * inv2RT;
    }
    __device__ __forceinline__ void invert_accel_z(const Vel& v, double dt, double geq, double Z, double vg,
                                                   double vb, double& gF, double& bF) const {
        double beq = (v.hx2 + cRT2) * geq;
        const double c = c2 * (v.ax - au);
        gF = geq + ig * (vg - geq + c * geq);
        bF = beq + ib * (vb - beq + 0.25 * dt * v.ax * (gF - geq) + c * beq) + eb * Z * (gF - geq);
    }
};

// ---------------------------------------------------------------------------
// Maxwellian by recurrence along the fastest velocity axis.  The nodes of
// velocity axis 0 are uniform (spacing h); with x_k = xi_k - u_x, s = 1/(2RT)
// and everything else fixed,
//   g_eq(k+1) = g_eq(k) R_k,  R_k = exp(-(2 x_k + h) h s),  R_{k+1} = R_k C,
//   C = exp(-2 h^2 s).
// g_eq and R are set from direct exponentials at every WALK-th node of axis 0
// (anchors; a row of the velocity grid starts with one), which bounds the
// rounding drift of the products to about WALK^2 ulp.  A block whose
// exponents could leave the range where the products stay normal numbers
// uses direct exponentials throughout.  The value at a node depends only on
// the node, not on where a velocity slice starts: a slice starting inside a
// block walks from that block's anchor.
// ---------------------------------------------------------------------------
constexpr int WALK = 8;

template <int D>
__device__ __forceinline__ double maxwellian(double A, double s, const double* u, const Vel& v) {
    double c2 = 0.0;
#pragma unroll
    for (int e = 0; e < D; ++e) {
        const double x = v.xi[e] - u[e];
        c2 += x * x;
    }
    return A * exp(-c2 * s);
}

// The Maxwellian at FP32 accuracy, for the update kernel of the FP32 storage
// forms (whose stored values carry a relative rounding of 2^-24): the exponent
// is split in FP64 as -|xi - u|^2 s log2(e) = n + f with n an integer and |f| <=
// 1/2; 2^f is the hardware FP32 base-2 exponential (within 1 ulp) of f rounded
// to FP32 (an argument error below 2^-25), and 2^n is applied exactly.  The
// relative error is below 1e-7, against about 1e-16 for the FP64 exponential
// at a quarter of the instructions.  Exponents below -1500 give 0.
// The exponent comes from Z = xi.u - |u|^2/2, which the face inversion and the
// S_b source need anyway: |xi - u|^2 = 2 (|xi|^2/2 - Z), so it takes one
// subtraction instead of D differences and squares.  The rounding of the
// expanded square (relative 1e-16 of |xi|^2 + |u|^2) stays far below the
// FP32 accuracy of the result.
__device__ __forceinline__ double maxwellian_f32z(double A, double s, double Z, double hx2) {
    const double t = fmax(2.0 * M_LOG2E * s * (Z - hx2), -1500.0);  // at most rounding above 0
    const double n = rint(t);
    return A * ldexp((double)__builtin_amdgcn_exp2f((float)(t - n)), (int)n);
}

struct GaussWalk {
    double E, R, C;
    bool ok;
    __device__ __forceinline__ void init(double s, double h) { C = exp(-2.0 * h * h * s); }
    // anchor at the current node (its axis-0 coordinate is v.xi[0])
    template <int D>
    __device__ __forceinline__ void anchor(double A, double s, const double* u, const Vel& v, double h) {
        const double x = v.xi[0] - u[0];
        E = maxwellian<D>(A, s, u, v);
        R = exp(-(x + x + h) * h * s);
        const double m = fmax(fabs(x), fabs(x + (WALK - 1) * h));
        ok = m * m * s < 600.0 && (m + m + h) * h * s < 600.0 && h * h * s < 300.0;
    }
    __device__ __forceinline__ void advance() {
        E *= R;
        R *= C;
    }
    template <int D>
    __device__ __forceinline__ double value(double A, double s, const double* u, const Vel& v) const {
        double geq = E;
        if (!ok) geq = maxwellian<D>(A, s, u, v);
        return geq;
    }
};

// ---------------------------------------------------------------------------
// face-sum kernel: for every velocity of the slice, phi_bar at the left face
// of each tile cell along each d (stored for the update kernel), and the
// velocity sums of the face (serial per thread, fixed order)
// ---------------------------------------------------------------------------
// DIR: the problem has Dirichlet sides; their ghost slots of the q box take
// the fixed states' equilibria (a separate instantiation keeps the register
// budget of the others unchanged).
// SS: the single-slope reconstruction option (stage 3 reads only the upwind
// cell's slopes).
// ACC: the problem has an external acceleration (stage 1 adds its source
// terms; the a = 0 instantiations keep their register budget).
// SUMS: the thread accumulates its faces' velocity sums over the slice;
// without, it stores the face values only (k_face_reduce sums them).
// SM: how the face values are stored (st_faces).
template <int D, typename ST, bool DIR = false, bool SS = false, int TID = 0, bool ACC = false, bool SUMS = true,
          int SM = fv_store_mode<D>()>
struct FaceSumKernel {
    using G = Geo<D, TID>;
    static constexpr int NT = G::NT;
    // every 2-D shape keeps the q-box slots and their Maxwellian recurrence
    // in registers (so the shape does not change a result)
    static_assert(D != 2 || G::CACHE_COEF, "2-D tile shapes must keep their q-box slots in registers");
    // stencil arithmetic (quarter-step values in LDS, limiters, face values) in
    // the storage precision; equilibria and the velocity sums stay FP64
    using CT = typename StoreT<ST>::C;
    using RT = typename StoreT<ST>::R;
    // q-box points per thread: slot 0 is the thread's own cell, the other
    // slots cover the halo
    static constexpr int NHALO = G::NQ - NT;
    static constexpr int NSLOT = 1 + (NHALO + NT - 1) / NT;

    // Box index of the h-th point of a box (extents BX, BY, BZ; the tile sits
    // at offsets OX, OY, OZ) that lies outside the tile, in box order: planes
    // below the tile in z are full, the tile's planes miss its TX x TY block,
    // and likewise rows within a plane.
    template <int BX, int BY, int OX, int OY, int OZ>
    __device__ static int ring_point(int h) {
        constexpr int PL = BX * BY;                 // points per full plane
        constexpr int PI = PL - G::TX * G::TY;      // ring points per tile plane
        constexpr int RI = BX - G::TX;              // ring points per tile row
        if (h < OZ * PL) return h;  // below the tile: box order equals ring order
        h -= OZ * PL;
        if (h >= G::TZ * PI) return (OZ + G::TZ) * PL + (h - G::TZ * PI);  // above
        const int z = OZ + h / PI;
        int rem = h % PI, y, x;
        if (rem < OY * BX) {
            y = rem / BX;
            x = rem % BX;
        } else {
            rem -= OY * BX;
            if (rem >= G::TY * RI) {
                rem -= G::TY * RI;
                y = OY + G::TY + rem / BX;
                x = rem % BX;
            } else {
                y = OY + rem / RI;
                const int c = rem % RI;
                x = c < OX ? c : c + G::TX;
            }
        }
        return x + BX * (y + BY * z);
    }
    __device__ static int halo_point(int h) { return ring_point<G::QX, G::QY, G::OQX, G::OQY, G::OQZ>(h); }
    __device__ static int slope_ring_point(int h) {
        return ring_point<G::AX, G::AY, G::OAX, G::OAY, G::OAZ>(h);
    }
    // slope-box points outside the tile, and passes over them
    static constexpr int NARING = G::NA - NT;
    static constexpr int NRING2 = (2 * NARING + NT - 1) / NT;  // (point, field) passes

    // With stored quarter-step fields (3-D) the q box is loaded; otherwise
    // it is computed from g, b and the cell coefficients of the q-box slots,
    // which every 1-D and 2-D shape keeps in registers.
    static constexpr bool QS = quarter_stored(D);
    static constexpr bool KQ = G::CACHE_COEF && !QS;
    static_assert(QS || KQ, "a tile shape must keep its q-box slot coefficients in registers");

    // 1-D and 2-D alternate two LDS buffers between consecutive velocities,
    // which removes the barrier that would otherwise end each velocity
    static constexpr int NBUF = D <= 2 ? 2 : 1;

    struct Smem {
        CT q[NBUF][2][G::NQ + 1];  // phi_bar_plus for g, b (entry NQ: unused slots)
        CT a[NBUF][2][D * G::NA];  // limited differences for g, b
    };

    __device__ static void run(const Problem& P, int tile, int slice, int nslices, Smem& sm) {
        const int tid = threadIdx.x;
        const long long N = P.N;
        int t = tile;
        const int ox = (t % P.tiles1[0]) * G::TX;
        t /= P.tiles1[0];
        const int oy = D >= 2 ? (t % P.tiles1[1]) * G::TY : 0;
        t /= P.tiles1[1];
        const int oz = D >= 3 ? t * G::TZ : 0;
        const int v0 = (int)((long long)P.V * slice / nslices);
        const int v1 = (int)((long long)P.V * (slice + 1) / nslices);

        // q-box points of this thread: slot 0 its own cell, then halo points
        // (halo enumerated in box order, interior skipped); source cell after
        // periodic wrap / outflow clamp
        // lq: box index in the low 20 bits; for a Dirichlet ghost, its side
        // 2 d + side plus one in the bits above (-1: unused slot)
        long long srcq[NSLOT];
        int lq[NSLOT];
        CellCoef kq[KQ ? NSLOT : 1];
        {
            int lx = tid % G::TX, ly = (tid / G::TX) % G::TY, lz = tid / (G::TX * G::TY);
            lq[0] = G::qidx(lx, ly, lz);
#pragma unroll
            for (int k = 1; k < NSLOT; ++k) {
                const int h = tid + (k - 1) * NT;  // halo ordinal
                lq[k] = h < NHALO ? halo_point(h) : -1;
            }
#pragma unroll
            for (int k = 0; k < NSLOT; ++k) {
                srcq[k] = 0;  // unused slots still load a valid address
                if (lq[k] < 0) continue;
                int r = lq[k];
                int rx = r % G::QX, ry = (r / G::QX) % G::QY, rz = r / (G::QX * G::QY);
                const int c3[3] = {ox + rx - G::OQX, oy + ry - G::OQY, oz + rz - G::OQZ};
                if constexpr (DIR) {
                    int side = 0;
#pragma unroll
                    for (int d = 0; d < D; ++d)
                        if (P.bc[d] == 2 && (c3[d] < 0 || c3[d] >= P.n[d])) side = 2 * d + (c3[d] >= P.n[d]) + 1;
                    lq[k] = r | (side << 20);
                }
                int cx = map_coord(c3[0], P.n[0], P.bc[0]);
                int cy = D >= 2 ? map_coord(c3[1], P.n[1], P.bc[1]) : 0;
                int cz = D >= 3 ? map_coord(c3[2], P.n[2], P.bc[2]) : 0;
                srcq[k] = cx + (long long)P.n[0] * (cy + (long long)P.n[1] * cz);
            }
            // every slot's coefficients, an unused slot's those of cell 0:
            // stage 1 evaluates each slot (its result unread for an unused one)
            if constexpr (KQ) {
#pragma unroll
                for (int k = 0; k < NSLOT; ++k) kq[k] = load_coef(P.P_in, N, srcq[k]);
            }
        }
        // own cell = the left faces this thread reconstructs
        const int tx = tid % G::TX, ty = (tid / G::TX) % G::TY, tz = tid / (G::TX * G::TY);
        const int gx = ox + tx, gy = oy + ty, gz = oz + tz;
        const long long NE = P.NE;
        long long fe = -1;  // extended-grid index of the own cell's left faces
        bool fvalid[D];
        {
            int cc[3] = {gx, gy, gz};
            bool any = false;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                bool ok = true;
#pragma unroll
                for (int e = 0; e < D; ++e) ok &= e == d ? cc[e] < P.ne[e] : cc[e] < P.n[e];
                fvalid[d] = ok;
                any |= ok;
            }
            if (any) fe = cc[0] + (long long)P.ne[0] * (cc[1] + (long long)P.ne[1] * cc[2]);
        }

        constexpr int NS = 2 * D + 3;
        double acc[SUMS ? D : 1][NS];
        if constexpr (SUMS) {
#pragma unroll
            for (int d = 0; d < D; ++d)
#pragma unroll
                for (int j = 0; j < NS; ++j) acc[d][j] = 0.0;
        }

        // Software pipelining: the next velocity's fields are loaded while the
        // current one is processed (when the q-box slots fit in registers).
        // The loop is unrolled by two over two named register sets, so a
        // register with a load in flight is never copied: a copy would make
        // the compiler wait for every outstanding memory operation, the face
        // value stores included.
        constexpr bool PREFETCH = NSLOT <= 2 || QS;
        const void* const src_g = QS ? P.qg : P.g_in;
        const void* const src_b = QS ? P.qb : P.b_in;
        RT pa_g[NSLOT], pa_b[NSLOT], pb_g[NSLOT], pb_b[NSLOT];
        if constexpr (PREFETCH) {
            load_slots<ST, NSLOT>(P, src_g, src_b, v0 < v1 ? v0 : 0, srcq, pa_g, pa_b);
        }
        const long long fstride = P.fv_stride;  // per (d, field) block of FV

        // Maxwellians of the q-box slots by recurrence along velocity axis 0
        // (when the slot coefficients live in registers)
        constexpr bool WALKER = KQ;
        const double h = P.hxi0;
        const int nvx = P.nv[0];
        GaussWalk wq[WALKER ? NSLOT : 1];
        if constexpr (WALKER) {
#pragma unroll
            for (int k = 0; k < NSLOT; ++k) wq[k].init(kq[k].inv2RT, h);
        }
        int ix = v0 % nvx;

        // one velocity: cur_* hold its prefetched fields, nxt_* receive the next
        auto velocity = [&](int i, int buf, RT(&cur_g)[NSLOT], RT(&cur_b)[NSLOT], RT(&nxt_g)[NSLOT],
                            RT(&nxt_b)[NSLOT]) __attribute__((always_inline)) {
            const Vel v = load_vel(P.vel, i);
            if constexpr (WALKER) {
                if (i == v0 || ix % WALK == 0) {
                    const int a0 = ix - ix % WALK;
                    const Vel va = a0 == ix ? v : load_vel(P.vel, i - (ix - a0));
#pragma unroll
                    for (int k = 0; k < NSLOT; ++k) wq[k].template anchor<D>(kq[k].A, kq[k].inv2RT, kq[k].u, va, h);
                    for (int j = a0; j < ix; ++j)
#pragma unroll
                        for (int k = 0; k < NSLOT; ++k) wq[k].advance();
                }
            }
            // BF16 rows: the raw halves move to the top of an FP32 word
            const bool half = StoreT<ST>::MIXED && (row_word(P, i) & 1);
            CT* const sq0 = sm.q[buf][0];
            CT* const sq1 = sm.q[buf][1];
            CT* const sa0 = sm.a[buf][0];
            CT* const sa1 = sm.a[buf][1];
            CT q_own[2], a_own[2][D];  // the own cell's q and slopes
            if constexpr (PREFETCH) {
                // unconditional loads (the last velocity re-reads itself) keep
                // the wait counts exact
                load_slots<ST, NSLOT>(P, src_g, src_b, i + 1 < v1 ? i + 1 : i, srcq, nxt_g, nxt_b);
            }

            // stage 1: quarter-step fields on the q box; a slot without a
            // point (the last ones of the halo) computes from cell 0 and
            // writes LDS entry NQ, which nothing reads, so the loop has no
            // branch between the loads of the previous velocity and their use
#pragma unroll
            for (int k = 0; k < NSLOT; ++k) {
                {
                    const int r = lq[k] >= 0 ? (lq[k] & 0xFFFFF) : G::NQ;
                    double g, b;
                    if constexpr (PREFETCH) {
                        g = slot_value<ST>(cur_g[k], half, srcq[k]);
                        b = slot_value<ST>(cur_b[k], half, srcq[k]);
                    } else {
                        g = state_ld<ST>(P, src_g, i, srcq[k]);
                        b = state_ld<ST>(P, src_b, i, srcq[k]);
                    }
                    double qg, qb;
                    if constexpr (QS) {
                        qg = g;
                        qb = b;
                    } else {
                        const double geq = wq[k].template value<D>(kq[k].A, kq[k].inv2RT, kq[k].u, v);
                        quarter_step_eq<D, ACC>(kq[k], v, geq, g, b, qg, qb, &P);
                    }
                    if constexpr (DIR) {
                        if (lq[k] > 0 && (lq[k] >> 20)) {  // Dirichlet ghost: the fixed state's equilibrium
                            const double* de = P.dir_eq + ((long long)((lq[k] >> 20) - 1) * P.V + i) * 2;
                            qg = de[0];
                            qb = de[1];
                        }
                    }
                    sq0[r] = CT(qg);
                    sq1[r] = CT(qb);
                    if (k == 0) {  // slot 0 is the own cell
                        q_own[0] = CT(qg);
                        q_own[1] = CT(qb);
                    }
                }
            }
            __syncthreads();

            // stage 2: limited differences on the slope box; the own cell first
            // (its values stay in registers for stage 3), then the ring
            {
                const int ai = G::aidx(tx, ty, tz), qi = G::qidx(tx, ty, tz);
#pragma unroll
                for (int e = 0; e < D; ++e) {
                    const int sq = G::SQ(e);
#pragma unroll
                    for (int f = 0; f < 2; ++f) {
                        const CT* q = f == 0 ? sq0 : sq1;
                        const CT c = q_own[f];
                        const CT a = half_van_leer(c - q[qi - sq], q[qi + sq] - c);
                        (f == 0 ? sa0 : sa1)[e * G::NA + ai] = a;
                        a_own[f][e] = a;
                    }
                }
            }
            // the ring: one (point, field) pair per thread and pass, so the
            // work spreads over all waves of the workgroup
#pragma unroll
            for (int k = 0; k < NRING2; ++k) {
                const int t = tid + k * NT;
                if (t < 2 * NARING) {
                    const int f = t >= NARING;
                    const int h = t - f * NARING;
                    const int p = slope_ring_point(h);
                    const int px = p % G::AX, py = (p / G::AX) % G::AY, pz = p / (G::AX * G::AY);
                    const int qi = (px + 1) + G::QX * ((py + (D >= 2 ? 1 : 0)) + G::QY * (pz + (D >= 3 ? 1 : 0)));
                    const CT* q = f == 0 ? sq0 : sq1;
                    CT* a = sa0 + f * (D * G::NA);
                    const CT c = q[qi];
#pragma unroll
                    for (int e = 0; e < D; ++e) {
                        const int sq = G::SQ(e);
                        a[e * G::NA + p] = half_van_leer(c - q[qi - sq], q[qi + sq] - c);
                    }
                }
            }
            __syncthreads();

            // stage 3: left face of the own cell along each d.  Upwind cell u
            // is c - d (xi_d > 0) or c (xi_d < 0); the own cell's q and slopes
            // come from registers, the others from LDS.
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int dxo = d == 0, dyo = d == 1, dzo = d == 2;
                const double xd = d == 0 ? v.xi[0] : (d == 1 ? v.xi[1] : v.xi[2]);
                const int q_m = G::qidx(tx - dxo, ty - dyo, tz - dzo);
                const int a_m = G::aidx(tx - dxo, ty - dyo, tz - dzo);
                const int a_mm = G::aidx(tx - 2 * dxo, ty - 2 * dyo, tz - 2 * dzo);
                const int a_p = G::aidx(tx + dxo, ty + dyo, tz + dzo);
                // Upwind side by the sign of xi_d, which is uniform across the
                // workgroup: tested on its bits with scalar integer
                // instructions, so each velocity takes one branch (the mean
                // of both one-sided values only for xi_d = 0).
                const long long xbits = __builtin_bit_cast(long long, xd);
                const bool from_left = xbits > 0;                               // xi_d > 0
                const bool from_right = xbits < 0 && (xbits << 1) != 0;          // xi_d < 0
                // the face value from the upwind cell c - d (left) or c (right)
                auto left_value = [&](int f) __attribute__((always_inline)) {
                    const CT* sq = f == 0 ? sq0 : sq1;
                    const CT* sa = f == 0 ? sa0 : sa1;
                    CT aU[D], aL[D], aR[D];
#pragma unroll
                    for (int e = 0; e < D; ++e) aU[e] = sa[e * G::NA + a_m];
                    if constexpr (SS) return face_value_single<D, CT>(sq[q_m], aU, d, CT(1), v);
                    // upwind c - d: its left and right neighbours are c - 2d and c
#pragma unroll
                    for (int e = 0; e < D; ++e) {
                        aL[e] = sa[e * G::NA + a_mm];
                        aR[e] = a_own[f][e];
                    }
                    return face_value_at<D, CT>(sq[q_m], aU, aL, aR, d, CT(1), v);
                };
                auto right_value = [&](int f) __attribute__((always_inline)) {
                    const CT* sa = f == 0 ? sa0 : sa1;
                    if constexpr (SS) return face_value_single<D, CT>(q_own[f], a_own[f], d, CT(-1), v);
                    // upwind c: neighbours c - d and c + d
                    CT aL[D], aR[D];
#pragma unroll
                    for (int e = 0; e < D; ++e) {
                        aL[e] = sa[e * G::NA + a_m];
                        aR[e] = sa[e * G::NA + a_p];
                    }
                    return face_value_at<D, CT>(q_own[f], a_own[f], aL, aR, d, CT(-1), v);
                };
                CT fv[2];
                if (from_left) {
                    fv[0] = left_value(0);
                    fv[1] = left_value(1);
                } else if (from_right) {
                    fv[0] = right_value(0);
                    fv[1] = right_value(1);
                } else {
                    fv[0] = CT(0.5) * (left_value(0) + right_value(0));
                    fv[1] = CT(0.5) * (left_value(1) + right_value(1));
                }
                const double vg = fv[0], vb2 = fv[1];
                {
                    // a face outside the grid goes to the row's spare element
                    // NE: with the store unconditional the compiler need not
                    // wait for it before using the next velocity's loads
                    const long long o =
                        (long long)(2 * d) * fstride + (long long)i * P.fv_pitch + (fvalid[d] ? fe : NE);
                    st_faces<CT, 2, SM>(P, o, fstride, fv);
                }
                if constexpr (SUMS) {
                    // weighted velocity products come from the table (uniform)
                    const const_dptr vp = vel_ptr(P.vel, i);
                    acc[d][0] += v.w * vg;
#pragma unroll
                    for (int e = 0; e < D; ++e) acc[d][1 + e] += vp[VE_WXI0 + e] * vg;
                    acc[d][D + 1] += v.w * vb2;
#pragma unroll
                    for (int e = 0; e < D; ++e) acc[d][D + 2 + e] += vp[VE_WXX + 3 * d + e] * vg;
                    acc[d][2 * D + 2] += vp[VE_WXI0 + d] * vb2;
                }
            }
            if constexpr (WALKER) {
#pragma unroll
                for (int k = 0; k < NSLOT; ++k) wq[k].advance();
                if (++ix == nvx) ix = 0;
            }
            // single-buffered: the next velocity must not overwrite q and a
            // before every thread has read them; double-buffered: the next
            // velocity writes the other buffer, and the one after that comes
            // only after two more barriers
            if constexpr (NBUF == 1) __syncthreads();
        };

        if constexpr (D <= 2) {
            // The first velocity is peeled off, so the loop is entered, like
            // its back edge, with a velocity's face-value stores in flight:
            // the compiler's wait counts at the loop head then need not wait
            // for those stores before the fields loaded ahead are used.
            int i = v0;
            if (i < v1) velocity(i++, 0, pa_g, pa_b, pb_g, pb_b);
            for (; i + 1 < v1; i += 2) {
                velocity(i, NBUF - 1, pb_g, pb_b, pa_g, pa_b);
                velocity(i + 1, 0, pa_g, pa_b, pb_g, pb_b);
            }
            if (i < v1) velocity(i, NBUF - 1, pb_g, pb_b, pa_g, pa_b);
        } else {
            // 3-D: registers allow one set; the copy costs a wait per velocity
            for (int i = v0; i < v1; ++i) {
                RT cg[NSLOT], cb[NSLOT];
#pragma unroll
                for (int k = 0; k < NSLOT; ++k) {
                    cg[k] = pa_g[k];
                    cb[k] = pa_b[k];
                }
                velocity(i, 0, cg, cb, pa_g, pa_b);
            }
        }

        // partial face sums of this velocity slice
        if constexpr (SUMS) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                if (!fvalid[d]) continue;
                double* out = P.FS + ((long long)(slice * D + d) * NS) * NE + fe;
#pragma unroll
                for (int j = 0; j < NS; ++j) out[(long long)j * NE] = acc[d][j];
            }
        }
    }
};

// ---------------------------------------------------------------------------
// cell closure: W^{n+1} = W^n - dt sum_d (G_right - G_left)/dx_d; coefs at n+1
// ---------------------------------------------------------------------------
// The left and right faces of cell c along each d (periodic wrap at the right
// end).  Cell and face indices fit 31 bits (checked at set-up).
template <int D>
__device__ __forceinline__ void cell_faces(const Problem& P, unsigned c, unsigned (&fl)[D], unsigned (&fr)[D]) {
    const unsigned n0 = P.n[0], n1 = P.n[1], e0 = P.ne[0], e1 = P.ne[1];
    const unsigned co[3] = {c % n0, D >= 2 ? (c / n0) % n1 : 0, D >= 3 ? c / (n0 * n1) : 0};
    const unsigned stride[3] = {1, e0, e0 * e1};
    const unsigned f = co[0] + e0 * (co[1] + e1 * co[2]);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const bool wrap = P.bc[d] == 0 && co[d] + 1 == (unsigned)P.n[d];
        fl[d] = f;
        fr[d] = wrap ? f - co[d] * stride[d] : f + stride[d];
    }
}

// Part of the single-problem update kernel: each of a cell's update threads
// (one per velocity slice) forms W^{n+1} and the coefficients it needs for
// itself, and the one of slice 0 (store) writes them for the next step.  The
// D + 2 flux moments of 2D faces are a few loads against hundreds of
// velocities, where a launch of its own cost 4 us of a 52 us step of the Sod
// tube and 13 us of 1.40 ms of the 256^2 x 28^2 step.  In the batched update
// the same code raised the FP32 2-D class from 165 to 231 registers (3 waves
// per SIMD to 2), so batches keep the launch (one for all problems, under 1%
// of their step).  fl, fr: the cell's left and right faces.
template <int D>
__device__ __forceinline__ CellCoef cell_close(const Problem& P, long long c, const unsigned (&fl)[D],
                                               const unsigned (&fr)[D], bool store) {
    const long long N = P.N, NE = P.NE;
    double Wn[D + 2], W0[D + 2];
#pragma unroll
    for (int k = 0; k < D + 2; ++k) W0[k] = Wn[k] = P.W_in[k * N + c];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const double* Gd = P.G + (long long)d * (D + 2) * NE;
#pragma unroll
        for (int k = 0; k < D + 2; ++k)
            Wn[k] -= P.dt * P.inv_dx[d] * (Gd[k * NE + fr[d]] - Gd[k * NE + fl[d]]);
    }
    if (P.has_accel) {
        // source integrals at t_n (eqs. rhouupdate, rhoEupdate): rho a, (rho u).a
#pragma unroll
        for (int e = 0; e < D; ++e) {
            Wn[1 + e] += P.dt * W0[0] * P.accel[e];
            Wn[D + 1] += P.dt * W0[1 + e] * P.accel[e];
        }
    }
    const Prim q = primitives(P, D, Wn);
    if (q.bad) raise_error(P.err);
    const CellCoef k = cell_coefs(P, D, q);
    if (store) {
#pragma unroll
        for (int e = 0; e < D + 2; ++e) P.W_out[e * N + c] = Wn[e];
        store_coef(P.P_out, N, c, k);
    }
    return k;
}

// ---------------------------------------------------------------------------
// update kernel: streaming, one thread per cell over a velocity slice.
// Reads phi^n and the stored phi_bar at the cell's 2D faces, inverts eq.
// phibar with the face coefficients, forms the microflux (eq. flux) and writes
// phi^{n+1} (eq. phiupdate).
// ---------------------------------------------------------------------------
// ACC: the problem has an external acceleration (face inversion, the cell
// source of eq. phiupdate and, in 3-D, the next quarter-step fields carry
// its terms).
// ROWS (BF16-tail form only): 0 updates every velocity row of the slice,
// 1 only its FP32 rows, 2 only its BF16 rows.  The 3-D single-problem step
// runs the two row kinds as two launches, so that each holds one loop body
// (see launch_update).
// CLOSE: the kernel closes its cells itself (cell_close); otherwise it loads
// the coefficients at n+1.
template <int D, typename ST, bool ACC = false, int ROWS = 0, bool CLOSE = true>
struct UpdateKernel {
    using CT = typename StoreT<ST>::C;  // stored face values
    __device__ static void run(const Problem& P, long long c, int slice, int nslices) {
        const long long N = P.N, NE = P.NE;
        const bool inside = c < N;
        const long long cc = inside ? c : 0;
        unsigned fl[D], fr[D];
        cell_faces<D>(P, (unsigned)cc, fl, fr);
        // Byte offsets of the cell and its faces in their rows: 32 bits reach
        // any row the device's memory can hold (checked at set-up), and a
        // uniform row plus a 32-bit offset is an address the loads and stores
        // form themselves, where 64-bit sums took 12 (2-D) and 18 (3-D) VALU
        // instructions per velocity.  A cell's left faces share one index.
        // (One set for g, one for b: of a shared one the sum with g's row would
        // be shared too, in 64 bits.)  Update of 64^3 x 16^3 FP32 13.9 -> 12.4
        // ms, 256^2 x 28^2 FP64 637 -> 629 us; the 2-D FP32 forms, which wait
        // for the rows' scalar arithmetic instead, lose (357 -> 372 us, batches
        // 5%) and keep the 64-bit sums.
        constexpr bool ROW32 = D != 2 || std::is_same<ST, double>::value;
        unsigned oc = (unsigned)cc, bl[2], br[2][D];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            bl[f] = fl[0] * (unsigned)sizeof(CT);
#pragma unroll
            for (int d = 0; d < D; ++d) br[f][d] = fr[d] * (unsigned)sizeof(CT);
        }
        auto store = [&](auto kind, void* base, long long off, double v) __attribute__((always_inline)) {
            using IO = RowIO<decltype(kind)>;
            if constexpr (ROW32) {
                unsigned ob = oc * (unsigned)IO::BYTES;
                keep_offset(ob);
                IO::st_at(base, off, ob, v);
            } else {
                IO::st(base, off, cc, v);
            }
        };
        const CellCoef k0 = load_coef(P.P_in, N, cc);
        CellCoef k1;
        if constexpr (CLOSE) k1 = cell_close<D>(P, cc, fl, fr, inside && slice == 0 && ROWS != 2);
        else k1 = load_coef(P.P_out, N, cc);
        FaceCoef<D> fcl[D], fcr[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const double* F = P.FP + (long long)d * NFP * NE;
            fcl[d].load(F + fl[d], NE);
            fcr[d].load(F + fr[d], NE);
            if constexpr (ACC) {
                fcl[d].prepare_accel(P.accel, P.dt);
                fcr[d].prepare_accel(P.accel, P.dt);
            }
        }
        // the cell's source terms at t_n: dt S_g = c0 g_eq, dt S_b = dt a.xi (g - g_eq) + c0 b_eq
        // with c0 = dt a.(xi - u)/(R T) = 2 dt (a.xi - a.u)/(2 R T)
        double au0 = 0.0;
        if constexpr (ACC) {
#pragma unroll
            for (int d = 0; d < D; ++d) au0 += P.accel[d] * k0.u[d];
        }
        const int v0 = (int)((long long)P.V * slice / nslices);
        const int v1 = (int)((long long)P.V * (slice + 1) / nslices);
        const long long fstride = P.fv_stride;
        const double dt = P.dt;
        // constant parts of eq. phiupdate
        const double inv_g = 1.0 / (1.0 + 2.0 * k1.beta), inv_b = 1.0 / (1.0 + 2.0 * k1.betab);

        // Maxwellians by recurrence along velocity axis 0 for FP64 storage in
        // 1-D and 2-D.  The 3-D kernel has no registers to spare, and the FP32
        // kernel runs a third wave per SIMD without the recurrence state,
        // which outweighs the exponentials it saves.
        constexpr bool WALKER = D <= 2 && std::is_same<ST, double>::value;
        const double h = P.hxi0;
        const int nvx = P.nv[0];
        GaussWalk w0, w1, wl[D], wr[D];
        if constexpr (WALKER) {
            w0.init(k0.inv2RT, h);
            w1.init(k1.inv2RT, h);
#pragma unroll
            for (int d = 0; d < D; ++d) {
                wl[d].init(fcl[d].inv2RT, h);
                wr[d].init(fcr[d].inv2RT, h);
            }
        }
        int ix = v0 % nvx;
        // Maxwellians without the recurrence: the FP64 exponential for FP64
        // storage; FP32 accuracy for the FP32 forms, from Z = xi.u - |u|^2/2,
        // which the inversion and the S_b source use as well
        constexpr bool FZ = !std::is_same<ST, double>::value;
        auto equilibrium = [](double A, double s, const double* u, double Z, const Vel& v)
                               __attribute__((always_inline)) {
            if constexpr (FZ) return maxwellian_f32z(A, s, Z, v.hx2);
            else return maxwellian<D>(A, s, u, v);
        };

        // The loads of one velocity: g and b of the cell, and the stored face
        // values at its 2D faces ([d][left g, left b, right g, right b]).
        auto load = [&](int i, long long off, auto kind, typename RowIO<decltype(kind)>::Raw& rg,
                        typename RowIO<decltype(kind)>::Raw& rb, CT (&fv)[4 * D]) __attribute__((always_inline)) {
            using IO = RowIO<decltype(kind)>;
            if constexpr (ROW32) {
                unsigned ob = oc * (unsigned)IO::BYTES;
                keep_offset(ob);
#pragma unroll
                for (int f = 0; f < 2; ++f) {
                    keep_offset(bl[f]);
#pragma unroll
                    for (int d = 0; d < D; ++d) keep_offset(br[f][d]);
                }
                rg = IO::raw_at(P.g_in, off, ob);
                rb = IO::raw_at(P.b_in, off, ob);
            } else {
                rg = IO::raw(P.g_in, off, cc);
                rb = IO::raw(P.b_in, off, cc);
            }
            const CT* const F = (const CT*)P.FV;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const CT* const rowg = F + ((long long)(2 * d) * fstride + (long long)i * P.fv_pitch);
                const CT* const rowb = rowg + fstride;
                if constexpr (ROW32) {
                    fv[4 * d] = at_byte(rowg, bl[0]);
                    fv[4 * d + 1] = at_byte(rowb, bl[1]);
                    fv[4 * d + 2] = at_byte(rowg, br[0][d]);
                    fv[4 * d + 3] = at_byte(rowb, br[1][d]);
                } else {
                    fv[4 * d] = rowg[fl[d]];
                    fv[4 * d + 1] = rowb[fl[d]];
                    fv[4 * d + 2] = rowg[fr[d]];
                    fv[4 * d + 3] = rowb[fr[d]];
                }
            }
        };
        // One velocity of the slice from its loads; its rows (g, b in and
        // out, and the 3-D quarter-step fields) hold elements of kind E and
        // start `off` bytes into each state array.  Every storage form runs
        // this one body.
        auto velocity = [&](int i, long long off, auto kind, const typename RowIO<decltype(kind)>::Raw& rg,
                            const typename RowIO<decltype(kind)>::Raw& rb, const CT (&fv)[4 * D])
                            __attribute__((always_inline)) {
            using IO = RowIO<decltype(kind)>;
            const Vel v = load_vel(P.vel, i);
            if constexpr (WALKER) {
                if (i == v0 || ix % WALK == 0) {
                    const int a0 = ix - ix % WALK;
                    // a slice starting inside a block walks from its anchor
                    const Vel va = a0 == ix ? v : load_vel(P.vel, i - (ix - a0));
                    w0.anchor<D>(k0.A, k0.inv2RT, k0.u, va, h);
                    w1.anchor<D>(k1.A, k1.inv2RT, k1.u, va, h);
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        wl[d].template anchor<D>(fcl[d].A, fcl[d].inv2RT, fcl[d].u, va, h);
                        wr[d].template anchor<D>(fcr[d].A, fcr[d].inv2RT, fcr[d].u, va, h);
                    }
                    for (int j = a0; j < ix; ++j) {
                        w0.advance();
                        w1.advance();
#pragma unroll
                        for (int d = 0; d < D; ++d) {
                            wl[d].advance();
                            wr[d].advance();
                        }
                    }
                }
            }
            const double g = IO::val(rg);
            const double b = IO::val(rb);
            double Fg = 0.0, Fb = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const double Zl = fcl[d].z(v), Zr = fcr[d].z(v);
                const double eql = WALKER ? wl[d].template value<D>(fcl[d].A, fcl[d].inv2RT, fcl[d].u, v)
                                          : equilibrium(fcl[d].A, fcl[d].inv2RT, fcl[d].u, Zl, v);
                const double eqr = WALKER ? wr[d].template value<D>(fcr[d].A, fcr[d].inv2RT, fcr[d].u, v)
                                          : equilibrium(fcr[d].A, fcr[d].inv2RT, fcr[d].u, Zr, v);
                double gl, bl, gr, br;
                const double flg = fv[4 * d], flb = fv[4 * d + 1], frg = fv[4 * d + 2], frb = fv[4 * d + 3];
                if constexpr (ACC) {
                    fcl[d].invert_accel_z(v, dt, eql, Zl, flg, flb, gl, bl);
                    fcr[d].invert_accel_z(v, dt, eqr, Zr, frg, frb, gr, br);
                } else {
                    fcl[d].invert_z(v, eql, Zl, flg, flb, gl, bl);
                    fcr[d].invert_z(v, eqr, Zr, frg, frb, gr, br);
                }
                const double sxd = v.xi[d] * P.inv_dx[d];
                Fg += sxd * (gr - gl);
                Fb += sxd * (br - bl);
            }
            double xu0 = 0.0, xu1 = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                xu0 += v.xi[d] * k0.u[d];
                xu1 += v.xi[d] * k1.u[d];
            }
            const double Z0 = xu0 - k0.hu2;
            const double geq0 =
                WALKER ? w0.value<D>(k0.A, k0.inv2RT, k0.u, v) : equilibrium(k0.A, k0.inv2RT, k0.u, Z0, v);
            const double beq0 = (v.hx2 + k0.cRT2) * geq0;
            const double geq1 = WALKER ? w1.value<D>(k1.A, k1.inv2RT, k1.u, v)
                                       : equilibrium(k1.A, k1.inv2RT, k1.u, xu1 - k1.hu2, v);
            const double beq1 = (v.hx2 + k1.cRT2) * geq1;
            // eq. phiupdate with dt/(2 tau) = 2 beta and dt S_b = 4 eta Z (g - g_eq)
            double gn = g + 2.0 * k1.beta * geq1 + 2.0 * k0.beta * (geq0 - g) - dt * Fg;
            double bn = b + 2.0 * k1.betab * beq1 + 2.0 * k0.betab * (beq0 - b) - dt * Fb +
                        4.0 * k0.eta * Z0 * (g - geq0);
            if constexpr (ACC) {
                const double c0 = 2.0 * dt * k0.inv2RT * (v.ax - au0);
                gn += c0 * geq0;
                bn += dt * v.ax * (g - geq0) + c0 * beq0;
            }
            gn *= inv_g;
            bn *= inv_b;
            if (inside) {
                store(kind, P.g_out, off, gn);
                store(kind, P.b_out, off, bn);
                if constexpr (quarter_stored(D)) {
                    // next step's phi_bar_plus from the state as stored
                    double qg, qb;
                    quarter_step_eq<D, ACC>(k1, v, geq1, IO::round(gn), IO::round(bn), qg, qb, &P);
                    store(kind, P.qg, off, qg);
                    store(kind, P.qb, off, qb);
                }
            }
            if constexpr (WALKER) {
                w0.advance();
                w1.advance();
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    wl[d].advance();
                    wr[d].advance();
                }
                if (++ix == nvx) ix = 0;
            }
        };

        auto off_of = [&](int i) { return (long long)i * P.pitch * (long long)sizeof(ST); };
        // FP64 in 1-D and 2-D has the registers to load a velocity ahead; the
        // FP32 forms would lose a wave per SIMD (2-D) or spill (3-D)
        constexpr bool AHEAD = std::is_same<ST, double>::value && D <= 2;
        if constexpr (!StoreT<ST>::MIXED && !AHEAD) {
            for (int i = v0; i < v1; ++i) {
                typename RowIO<ST>::Raw rg, rb;
                CT fv[4 * D];
                load(i, off_of(i), ST{}, rg, rb, fv);
                // every load before any of the arithmetic (3-D FP64; left to
                // itself the compiler sinks some, 690 -> 661 us on 37 x 29 x 23
                // cells x 11 x 10 x 12; FP32 gains nothing).  Not in batches
                // without an acceleration, whose two waves per SIMD it costs
                // spills (four of 32^3 x 8^3: 1441 us with it, 1370 without;
                // with an acceleration, one wave, 6.2 and 8.3 ms per step)
                if constexpr (std::is_same<ST, double>::value && (CLOSE || ACC)) __builtin_amdgcn_sched_barrier(1);
                velocity(i, off_of(i), ST{}, rg, rb, fv);
            }
        } else if constexpr (!StoreT<ST>::MIXED) {
            // The loads of velocity i+1 are issued before velocity i is
            // processed, into the other of two named register sets (the loop
            // is unrolled by two), so a register with a load in flight is
            // never copied; the last trip re-reads its own velocity.
            typename RowIO<ST>::Raw ga, ba, gb, bb;
            CT fa[4 * D], fb[4 * D];
            if (v0 < v1) load(v0, off_of(v0), ST{}, ga, ba, fa);
            int i = v0;
            for (; i + 1 < v1; i += 2) {
                load(i + 1, off_of(i + 1), ST{}, gb, bb, fb);
                velocity(i, off_of(i), ST{}, ga, ba, fa);
                const int n2 = i + 2 < v1 ? i + 2 : i + 1;
                load(n2, off_of(n2), ST{}, ga, ba, fa);
                velocity(i + 1, off_of(i + 1), ST{}, gb, bb, fb);
            }
            if (i < v1) velocity(i, off_of(i), ST{}, ga, ba, fa);
        } else {
            // BF16-tail form: the row kind is uniform, so each velocity runs
            // the body for FP32 or BF16 rows; the FP32 rows of the slice
            // first, then its BF16 rows (every (cell, velocity) is updated on
            // its own, so the order is free); no recurrence for the equilibria
            if constexpr (ROWS != 2) {
                for (int i = v0; i < v1; ++i) {
                    const long long o = row_word(P, i);
                    if (!(o & 1)) {
                        float rg, rb;
                        CT fv[4 * D];
                        load(i, o, float{}, rg, rb, fv);
                        velocity(i, o, float{}, rg, rb, fv);
                    }
                }
            }
            if constexpr (ROWS != 1) {
                for (int i = v0; i < v1; ++i) {
                    const long long o = row_word(P, i);
                    if (o & 1) {
                        __bf16 rg, rb;
                        CT fv[4 * D];
                        load(i, o & ~1LL, Bf16Row{}, rg, rb, fv);
                        velocity(i, o & ~1LL, Bf16Row{}, rg, rb, fv);
                    }
                }
            }
        }
    }
};

// waves per SIMD the face-sum kernel is compiled for (register budget; 3-D
// takes what it needs, within what a workgroup of its shape requires)
template <int D>
constexpr int face_sum_waves() { return D == 1 ? 4 : (D == 2 ? 3 : 1); }

// The single-problem face-sum kernel of tile shape TID.
template <int D, typename ST, bool DIR, bool SS, int TID, bool ACC, bool SUMS = true, int SM = fv_store_mode<D>()>
__global__ __launch_bounds__(tile_threads(D, TID), face_sum_waves<D>()) void k_face_sums(Problem P) {
    using K = FaceSumKernel<D, ST, DIR, SS, TID, ACC, SUMS, SM>;
    static_assert(sizeof(typename K::Smem) == face_sum_lds_bytes(D, TID, sizeof(typename K::CT)),
                  "host and kernel LDS sizes differ");
    __shared__ typename K::Smem sm;
    int ntiles = P.tiles1[0] * P.tiles1[1] * P.tiles1[2];
    int q = xcd_remap(blockIdx.x, gridDim.x);
    K::run(P, q % ntiles, q / ntiles, SUMS ? P.nslices : P.value_slices, sm);
}

// Velocity sums of the stored face values of one velocity slice: per face
// along d, the 2D+3 sums of the box kernel with the same products in the same
// ascending-velocity order, so the partial sums are bitwise those the box
// kernel accumulates in registers.  One thread per face-grid point takes its
// D faces.
template <int D, typename CT, int TB, int UNROLL>
__global__ __launch_bounds__(TB) void k_face_reduce(Problem P) {
    const long long fe = (long long)blockIdx.x * TB + threadIdx.x;
    const int slice = blockIdx.y;
    if (fe >= P.NE) return;
    const int c[3] = {(int)(fe % P.ne[0]), (int)((fe / P.ne[0]) % P.ne[1]),
                      (int)(fe / ((long long)P.ne[0] * P.ne[1]))};
    bool valid[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        bool ok = true;
#pragma unroll
        for (int e = 0; e < D; ++e) ok &= e == d ? c[e] < P.ne[e] : c[e] < P.n[e];
        valid[d] = ok;
    }
    const int v0 = (int)((long long)P.V * slice / P.nslices);
    const int v1 = (int)((long long)P.V * (slice + 1) / P.nslices);
    constexpr int NS = 2 * D + 3;
    double acc[D][NS];
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
        for (int j = 0; j < NS; ++j) acc[d][j] = 0.0;
    const CT* const fv = (const CT*)P.FV + fe;
#pragma unroll UNROLL
    for (int i = v0; i < v1; ++i) {
        const Vel v = load_vel(P.vel, i);
        const const_dptr vp = vel_ptr(P.vel, i);
        const long long row = (long long)i * P.fv_pitch;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            // invalid faces read a stored slot of the block and discard it
            const double vg = fv[(long long)(2 * d) * P.fv_stride + row];
            const double vb2 = fv[(long long)(2 * d + 1) * P.fv_stride + row];
            acc[d][0] += v.w * vg;
#pragma unroll
            for (int e = 0; e < D; ++e) acc[d][1 + e] += vp[VE_WXI0 + e] * vg;
            acc[d][D + 1] += v.w * vb2;
#pragma unroll
            for (int e = 0; e < D; ++e) acc[d][D + 2 + e] += vp[VE_WXX + 3 * d + e] * vg;
            acc[d][2 * D + 2] += vp[VE_WXI0 + d] * vb2;
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
        if (!valid[d]) continue;
        double* out = P.FS + ((long long)(slice * D + d) * NS) * P.NE + fe;
#pragma unroll
        for (int j = 0; j < NS; ++j) out[(long long)j * P.NE] = acc[d][j];
    }
}

template <int D, typename CT>
hipError_t launch_face_reduce(const Problem& P, hipStream_t s) {
    if constexpr (D <= 2) {
        // few threads and long sums: single waves spread over the CUs, and
        // enough velocities' values in flight to cover their latency
        constexpr int TB = 64;
        hipLaunchKernelGGL((k_face_reduce<D, CT, TB, D == 1 ? 16 : 8>), dim3((unsigned)((P.NE + TB - 1) / TB), P.nslices),
                           dim3(TB), 0, s, P);
    } else {
        hipLaunchKernelGGL((k_face_reduce<D, CT, WG, 4>), dim3((unsigned)((P.NE + WG - 1) / WG), P.nslices), dim3(WG), 0,
                           s, P);
    }
    return hipGetLastError();
}

// Launch the face sums of a problem of dimension D: the kernel of its tile
// shape, storage form, boundary kind and reconstruction.  Shapes whose boxes
// do not fit a CU's LDS for the storage form are refused (the host never
// selects them).
template <int D, typename ST, bool DIR, bool SS, int TID, bool ACC = false>
hipError_t launch_face_sums_shape(const Problem& P, hipStream_t s) {
    if constexpr (face_tile_fits(D, TID, sizeof(typename StoreT<ST>::C))) {
        const unsigned nt = (unsigned)(P.tiles1[0] * P.tiles1[1] * P.tiles1[2]);
        if constexpr (D <= 2 && TID == 0) {
            if (P.value_slices > 0) {
                hipLaunchKernelGGL((k_face_sums<D, ST, DIR, SS, TID, ACC, false>), dim3(nt * P.value_slices),
                                   dim3(tile_threads(D, TID)), 0, s, P);
                hipError_t e = hipGetLastError();
                if (e != hipSuccess) return e;
                return launch_face_reduce<D, typename StoreT<ST>::C>(P, s);
            }
        }
        if constexpr (D == 2 && (TID == 0 || std::is_same<ST, double>::value)) {
            if (P.fv_stream) {
                hipLaunchKernelGGL((k_face_sums<D, ST, DIR, SS, TID, ACC, true, FV_STREAM>), dim3(nt * P.nslices),
                                   dim3(tile_threads(D, TID)), 0, s, P);
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((k_face_sums<D, ST, DIR, SS, TID, ACC>), dim3(nt * P.nslices), dim3(tile_threads(D, TID)), 0,
                           s, P);
        return hipGetLastError();
    } else {
        return hipErrorInvalidConfiguration;
    }
}

template <int D, typename ST, int TID>
int face_sum_occupancy_shape() {
    if constexpr (face_tile_fits(D, TID, sizeof(typename StoreT<ST>::C))) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (k_face_sums<D, ST, false, false, TID, false>),
                                                        tile_threads(D, TID), 0) != hipSuccess) {
            (void)hipGetLastError();
            return 0;
        }
        return n;
    } else {
        return 0;
    }
}

// ---------------------------------------------------------------------------
// 3-D face values by z-march (the tile shapes with z = 0).  A workgroup owns a
// TX x TY column of the face grid for one velocity i and walks it along z.
// Step z stages the quarter-step fields of plane z+2 (with the xy halo,
// offsets -3..T+1), forms the limited differences of plane z+1 (all three
// components, offsets -2..T) and reconstructs the three left faces of its
// cells in plane z with the box kernel's operands and operations, so the face
// values are bitwise those of the box kernel.  LDS holds the q planes
// z-1..z+2 in a ring of four and the differences of planes z and z+1 in a
// ring of two; the own column's differences of planes z-2 and z-1 and its q
// of plane z-1 stay in registers.  Each plane is staged once per column
// (plus the xy halo), where a box stages (T_z + 5) planes per T_z.
// Two barriers per step keep the rings safe: the q store of step z goes to
// the slot of plane z-2, whose last reader is step z-1's differences (before
// that step's second barrier); the differences of step z go to the slot of
// plane z-1, whose last reader is step z-1's faces (before step z's first
// barrier).
// NF threads per cell: with NF = 2 (FP64, whose LDS allows two workgroups per
// CU) one thread per cell takes g and another b, which doubles the waves that
// hide the LDS and memory latency; with NF = 1 a thread takes both fields.
// The kernel stores the face values only; k_face_reduce forms their velocity
// sums.
template <typename CT>
constexpr int zmarch_threads_per_cell() { return sizeof(CT) == 8 ? 2 : 1; }

// TX = 0: the column is P.column[0] x P.column[1] cells, up to TY of them,
// chosen for the problem's extents within the bounds of column_fits, and the
// workgroup one wave per 64 cells and thread of a cell.  (Against 16 x 16
// columns of the same number: 48 x 40 x 24 FP64 1695 and 1683 us.)
template <typename ST, bool DIR, bool SS, int TX, int TY>
struct ZMarch {
    using CT = typename StoreT<ST>::C;
    using RT = typename StoreT<ST>::R;
    static constexpr bool FIXED = TX > 0;
    static constexpr int NT = FIXED ? TX * TY : TY;           // cells of the column (at most)
    static constexpr int NF = zmarch_threads_per_cell<CT>();  // threads per cell
    static constexpr int NTH = NF * NT;                       // threads of the workgroup (at most)
    static constexpr int FL = 2 / NF;                         // fields per thread
    // points of a q plane and of a difference plane (at most)
    static constexpr int NQ = FIXED ? (TX + 5) * (TY + 5) : column_nq(TY);
    static constexpr int NA = FIXED ? (TX + 3) * (TY + 3) : column_na(TY);
    static constexpr int NSLOT = FIXED ? (NQ + NT - 1) / NT : COLUMN_SLOTS;  // q points per thread
    // (point, field) passes
    static constexpr int NPASS = FIXED ? (2 * NA + NTH - 1) / NTH : column_passes(NF);
    static_assert(NF == 1 || !StoreT<ST>::MIXED, "the BF16-tail form loads its rows through load_slots");
    struct Smem {
        CT q[4][2][NQ];
        CT a[2][2][3][NA];  // [ring][field][component][point]
    };

    __device__ static void run(const Problem& P, int tile, int i, Smem& sm) {
        const int tx0 = FIXED ? TX : P.column[0], ty0 = FIXED ? TY : P.column[1];
        const int QX = tx0 + 5, nq = QX * (ty0 + 5);
        const int AX = tx0 + 3, na = AX * (ty0 + 3);
        const int nth = FIXED ? NTH : (int)blockDim.x;
        const int nt = FIXED ? NT : nth / NF;  // threads per field, whole waves
        auto qidx = [&](int x, int y) __attribute__((always_inline)) { return (x + 3) + QX * (y + 3); };
        auto aidx = [&](int x, int y) __attribute__((always_inline)) { return (x + 2) + AX * (y + 2); };
        const int tid = threadIdx.x;
        // first field of the thread (uniform per wave) and cell of the column
        const int f0 = NF == 2 ? (FIXED ? tid / NT : tid >= nt) : 0;
        const int ct = FIXED ? tid % NT : tid - f0 * nt;
        const int ox = (tile % P.tiles1[0]) * tx0, oy = (tile / P.tiles1[0]) * ty0;
        const int n0 = P.n[0], n1 = P.n[1], n2 = P.n[2];
        const long long nplane = (long long)n0 * n1;
        // q-plane points of this thread: in-plane source offset after the
        // periodic wrap / outflow clamp, and for Dirichlet sides the side of
        // the point's x or y coordinate (2 d + side + 1, y over x, 0: none)
        unsigned off[NSLOT];
        int lq[NSLOT];
        int sxy[DIR ? NSLOT : 1];
#pragma unroll
        for (int k = 0; k < NSLOT; ++k) {
            const int p = ct + k * nt;
            lq[k] = p < nq ? p : -1;
            const int pp = p < nq ? p : 0;
            const int x = ox + pp % QX - 3, y = oy + pp / QX - 3;
            off[k] = (unsigned)map_coord(x, n0, P.bc[0]) + (unsigned)n0 * (unsigned)map_coord(y, n1, P.bc[1]);
            if constexpr (DIR) {
                int side = 0;
                if (P.bc[0] == 2 && (x < 0 || x >= n0)) side = (x >= n0) + 1;
                if (P.bc[1] == 2 && (y < 0 || y >= n1)) side = 2 + (y >= n1) + 1;
                sxy[k] = side;
            }
        }
        const Vel v = load_vel(P.vel, i);
        const bool half = StoreT<ST>::MIXED && (row_word(P, i) & 1);

        // raw fields of the next plane to stage: both, or the thread's one
        RT pg[NSLOT], pb[NSLOT];
        auto load_plane = [&](int z) __attribute__((always_inline)) {
            const long long base = (long long)map_coord(z, n2, P.bc[2]) * nplane;
            if constexpr (StoreT<ST>::MIXED) {
                long long src[NSLOT];
#pragma unroll
                for (int k = 0; k < NSLOT; ++k) src[k] = base + off[k];
                load_slots<ST, NSLOT, false>(P, P.qg, P.qb, i, src, pg, pb);
            } else {
                // the plane's start is uniform, a point's offset in it 32 bits
                const ST* const rg = (const ST*)(f0 ? P.qb : P.qg) + ((long long)i * P.pitch + base);
                const ST* const rb = (const ST*)P.qb + ((long long)i * P.pitch + base);
#pragma unroll
                for (int k = 0; k < NSLOT; ++k) {
                    unsigned o = off[k] * (unsigned)sizeof(ST);
                    keep_offset(o);
                    pg[k] = at_byte(rg, o);
                    if constexpr (NF == 1) pb[k] = at_byte(rb, o);
                }
            }
        };
        auto store_plane = [&](int z) __attribute__((always_inline)) {
            const int r = (z + 8) & 3;
            int zs = 0;  // Dirichlet side of the plane (z over x and y)
            if constexpr (DIR) {
                if (P.bc[2] == 2 && (z < 0 || z >= n2)) zs = 4 + (z >= n2) + 1;
            }
#pragma unroll
            for (int k = 0; k < NSLOT; ++k) {
                if (lq[k] < 0) continue;
#pragma unroll
                for (int j = 0; j < FL; ++j) {
                    const int f = f0 + j;
                    double val = slot_value<ST>(j == 0 ? pg[k] : pb[k], half, 0);
                    if constexpr (DIR) {
                        const int side = zs ? zs : sxy[k];
                        if (side) val = P.dir_eq[((long long)(side - 1) * P.V + i) * 2 + f];
                    }
                    sm.q[r][f][lq[k]] = CT(val);
                }
            }
        };
        // limited differences of plane z on the difference plane
        int dq[NPASS], da[NPASS];  // a pass's points in a q plane's and a difference plane's two fields
#pragma unroll
        for (int k = 0; k < NPASS; ++k) {
            const int t = tid + k * nth;
            const int f = t >= na;
            const int pt = t - f * na;
            dq[k] = f * NQ + (pt % AX + 1) + QX * (pt / AX + 1);
            da[k] = f * 3 * NA + pt;
        }
        auto differences = [&](int z) __attribute__((always_inline)) {
            const int rm = (z + 7) & 3, r0 = (z + 8) & 3, rp = (z + 9) & 3, ra = (z + 8) & 1;
#pragma unroll
            for (int k = 0; k < NPASS; ++k) {
                if (tid + k * nth < 2 * na) {
                    const CT *q = sm.q[r0][0] + dq[k], *qm = sm.q[rm][0] + dq[k], *qp = sm.q[rp][0] + dq[k];
                    CT* const a = sm.a[ra][0][0] + da[k];
                    const CT c = q[0];
                    a[0] = half_van_leer(c - q[-1], q[1] - c);
                    a[NA] = half_van_leer(c - q[-QX], q[QX] - c);
                    a[2 * NA] = half_van_leer(c - qm[0], qp[0] - c);
                }
            }
        };

        // own cell, the validity of its left faces and their face-grid index
        // (a thread past the last cell takes cell 0 and no valid face)
        const bool own = FIXED || ct < tx0 * ty0;
        const int cc = own ? ct : 0;
        const int tx = cc % tx0, ty = cc / tx0;
        const int gx = ox + tx, gy = oy + ty;
        const bool vx = own && gx < P.ne[0] && gy < n1, vy = own && gx < n0 && gy < P.ne[1],
                   vz = own && gx < n0 && gy < n1;
        const unsigned fplane = (unsigned)P.ne[0] * (unsigned)P.ne[1], spare = (unsigned)P.NE;
        const unsigned fe0 = (unsigned)gx + (unsigned)P.ne[0] * (unsigned)gy;
        const long long fstride = P.fv_stride;
        const int qo_i = qidx(tx, ty), ao_i = aidx(tx, ty);

        // own column, per field of the thread: differences of planes z-2 and
        // z-1, q of plane z-1
        CT am2[FL][3], am1[FL][3], qm1[FL];
        auto faces = [&](int z, bool emit) __attribute__((always_inline)) {
            const int rq = (z + 8) & 3, ra = (z + 8) & 1, ra1 = (z + 9) & 1;
            CT qo[FL], ao[FL][3];
#pragma unroll
            for (int j = 0; j < FL; ++j) {
                qo[j] = sm.q[rq][f0 + j][qo_i];
#pragma unroll
                for (int e = 0; e < 3; ++e) ao[j][e] = sm.a[ra][f0 + j][e][ao_i];
            }
            if (emit) {
                const unsigned fe = fe0 + fplane * (unsigned)z;  // 32 bits hold a row (checked at set-up)
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const bool valid = d == 0 ? (vx && z < n2) : (d == 1 ? (vy && z < n2) : vz);
                    const int dx = d == 0, dy = d == 1;
                    const int a_m = aidx(tx - dx, ty - dy), a_mm = aidx(tx - 2 * dx, ty - 2 * dy);
                    const int a_p = aidx(tx + dx, ty + dy), q_m = qidx(tx - dx, ty - dy);
                    // the face value from the upwind cell c - d (left) or c
                    // (right), for field slot j of the thread
                    auto left_value = [&](int j) __attribute__((always_inline)) {
                        const int f = f0 + j;
                        CT qU, aU[3], aL[3];
                        if (d == 2) {
                            qU = qm1[j];
#pragma unroll
                            for (int e = 0; e < 3; ++e) {
                                aU[e] = am1[j][e];
                                aL[e] = am2[j][e];
                            }
                        } else {
                            qU = sm.q[rq][f][q_m];
#pragma unroll
                            for (int e = 0; e < 3; ++e) {
                                aU[e] = sm.a[ra][f][e][a_m];
                                aL[e] = sm.a[ra][f][e][a_mm];
                            }
                        }
                        if constexpr (SS) return face_value_single<3, CT>(qU, aU, d, CT(1), v);
                        return face_value_at<3, CT>(qU, aU, aL, ao[j], d, CT(1), v);
                    };
                    auto right_value = [&](int j) __attribute__((always_inline)) {
                        const int f = f0 + j;
                        if constexpr (SS) return face_value_single<3, CT>(qo[j], ao[j], d, CT(-1), v);
                        CT aL[3], aR[3];
#pragma unroll
                        for (int e = 0; e < 3; ++e) {
                            aL[e] = d == 2 ? am1[j][e] : sm.a[ra][f][e][a_m];
                            aR[e] = d == 2 ? sm.a[ra1][f][e][ao_i] : sm.a[ra][f][e][a_p];
                        }
                        return face_value_at<3, CT>(qo[j], ao[j], aL, aR, d, CT(-1), v);
                    };
                    // upwind side by the bits of the uniform xi_d, as in the
                    // box kernel
                    const long long xbits = __builtin_bit_cast(long long, v.xi[d]);
                    const bool from_left = xbits > 0;
                    const bool from_right = xbits < 0 && (xbits << 1) != 0;
                    CT fv[FL];
                    if (from_left) {
#pragma unroll
                        for (int j = 0; j < FL; ++j) fv[j] = left_value(j);
                    } else if (from_right) {
#pragma unroll
                        for (int j = 0; j < FL; ++j) fv[j] = right_value(j);
                    } else {
#pragma unroll
                        for (int j = 0; j < FL; ++j) fv[j] = CT(0.5) * (left_value(j) + right_value(j));
                    }
                    {
                        // a face outside the grid goes to the row's spare
                        // element NE (the store stays unconditional)
                        CT* const row = (CT*)P.FV + ((long long)(2 * d + f0) * fstride + (long long)i * P.fv_pitch);
                        st_faces_row<CT, FL, FV_EITHER>(P, row, (valid ? fe : spare) * (unsigned)sizeof(CT), fstride,
                                                        fv);
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < FL; ++j) {
                qm1[j] = qo[j];
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    am2[j][e] = am1[j][e];
                    am1[j][e] = ao[j][e];
                }
            }
        };

        // Planes z0-3 and z0-2 first; then step z stages plane z+2 (loaded
        // during the previous step), loads plane z+3, forms the differences of
        // plane z+1 and, from z0 on, the faces of plane z.  The steps before
        // z0 only fill the rings and the column registers (the differences of
        // plane z0-3 they shift through are never used).  The last step's
        // load of a plane past the column reads a mapped, valid address.
        const int z0 = 0, z1 = P.ne[2];
        load_plane(z0 - 3);
        store_plane(z0 - 3);
        load_plane(z0 - 2);
        store_plane(z0 - 2);
        load_plane(z0 - 1);
        for (int z = z0 - 3; z < z1; ++z) {
            store_plane(z + 2);
            load_plane(z + 3);
            __syncthreads();
            differences(z + 1);
            __syncthreads();
            faces(z, z >= z0);
        }
    }
};

template <typename ST, bool DIR, bool SS, int TX, int TY>
__global__ __launch_bounds__((ZMarch<ST, DIR, SS, TX, TY>::NTH)) void k_face_values_z(Problem P) {
    using K = ZMarch<ST, DIR, SS, TX, TY>;
    __shared__ typename K::Smem sm;
    const int ntiles = P.tiles1[0] * P.tiles1[1];
    const int q = xcd_remap(blockIdx.x, gridDim.x);
    K::run(P, q % ntiles, q / ntiles, sm);
}

// Face values by z-march, then their velocity sums (tile shape TID with z = 0).
template <typename ST, bool DIR, bool SS, int TID>
hipError_t launch_face_sums_zmarch(const Problem& P, hipStream_t s) {
    constexpr TileExt T = tile_shape(3, TID);
    static_assert(tile_zmarch(3, TID), "not a z-marching shape");
    using K = ZMarch<ST, DIR, SS, T.x, T.y>;
    static_assert(sizeof(typename K::Smem) == face_sum_lds_bytes(3, TID, sizeof(typename K::CT)),
                  "host and kernel LDS sizes differ");
    if constexpr (face_tile_fits(3, TID, sizeof(typename K::CT))) {
        const unsigned nb = (unsigned)((long long)P.tiles1[0] * P.tiles1[1] * P.V);
        if (P.column[0] > 0) {
            const dim3 block(K::NF * 64u * ((unsigned)(P.column[0] * P.column[1] + 63) / 64));
            if (column_fits(P.column[0], P.column[1], K::NF, 192))
                hipLaunchKernelGGL((k_face_values_z<ST, DIR, SS, 0, 192>), dim3(nb), block, 0, s, P);
            else if (column_fits(P.column[0], P.column[1], K::NF, 256))
                hipLaunchKernelGGL((k_face_values_z<ST, DIR, SS, 0, 256>), dim3(nb), block, 0, s, P);
            else
                return hipErrorInvalidConfiguration;
        } else {
            hipLaunchKernelGGL((k_face_values_z<ST, DIR, SS, T.x, T.y>), dim3(nb), dim3(K::NTH), 0, s, P);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_face_reduce<3, typename K::CT>(P, s);
    } else {
        return hipErrorInvalidConfiguration;
    }
}

template <typename ST, int TID>
int face_values_z_occupancy() {
    constexpr TileExt T = tile_shape(3, TID);
    if constexpr (face_tile_fits(3, TID, sizeof(typename StoreT<ST>::C))) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (k_face_values_z<ST, false, false, T.x, T.y>),
                                                        ZMarch<ST, false, false, T.x, T.y>::NTH, 0) != hipSuccess) {
            (void)hipGetLastError();
            return 0;
        }
        return n;
    } else {
        return 0;
    }
}

// Batched face sums: one launch for every tile of every problem of a storage
// class.  Persistent: the grid covers the resident slots and the workgroups
// take (cost-sorted, largest first) items from a device queue: an atomic
// counter, so a workgroup that finishes early takes the next item.  Which
// workgroup computes an item does not change its result.  The launch resets
// the other kernel's counter (that kernel's previous launch has finished and
// its next one starts after this one), so no memset enters a graph.
// Problems of different dimension share the launch; LDS is the union of their
// needs.
// The item index is uniform across the workgroup; readfirstlane tells the
// compiler so, and the item and its problem descriptor are then read through
// the constant address space: scalar loads into SGPRs instead of a copy of
// the descriptor in vector registers (the FP32 1-D/2-D face-sum class then
// runs 3 waves per SIMD, like the single-problem kernel).  Forcing the update
// class to 3 waves as well spills registers and is slower.
__device__ __forceinline__ int next_item(int* queue, int* slot) {
    if (threadIdx.x == 0) *slot = atomicAdd(queue, 1);
    __syncthreads();
    const int w = __builtin_amdgcn_readfirstlane(*slot);
    __syncthreads();  // every thread has read the slot before it is refilled
    return w;
}

// word-wise copy of a uniform descriptor through the constant address space
template <typename T>
__device__ __forceinline__ T load_uniform(const T* p) {
    static_assert(sizeof(T) % 4 == 0, "descriptor size");
    typedef const __attribute__((address_space(4))) unsigned* const_uptr;
    const const_uptr s = (const_uptr)(const void*)p;
    unsigned words[sizeof(T) / 4];
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); ++k) words[k] = s[k];
    T r;
    __builtin_memcpy(&r, words, sizeof(T));
    return r;
}

// ---------------------------------------------------------------------------
// face closure: W_f, coefficients, flux moments
// ---------------------------------------------------------------------------
// Whether face f (extended-grid index) with normal d lies in the grid.
template <int D>
__device__ __forceinline__ bool face_in_grid(const Problem& P, int d, unsigned f) {
    const unsigned ne0 = P.ne[0], ne1 = P.ne[1];
    const unsigned cc[3] = {f % ne0, D >= 2 ? (f / ne0) % ne1 : 0, D >= 3 ? f / (ne0 * ne1) : 0};
    bool in = true;
#pragma unroll
    for (int e = 0; e < D; ++e) in &= cc[e] < (unsigned)P.n[e] || (e == d && P.bc[e] != 0);
    return in;
}

// W_f from the face's velocity sums S, and its primitives.
template <int D>
__device__ __forceinline__ Prim face_primitives(const Problem& P, const double (&S)[2 * D + 3]) {
    double Wf[D + 2];
#pragma unroll
    for (int j = 0; j < D + 2; ++j) Wf[j] = S[j];
    if (P.has_accel) {
        // eqs. rhoubar, rhoEbar: (h/2) rho a and (h/2) (rho u).a, h/2 = dt/4,
        // with the face momentum just formed
#pragma unroll
        for (int e = 0; e < D; ++e) Wf[1 + e] += 0.25 * P.dt * Wf[0] * P.accel[e];
#pragma unroll
        for (int e = 0; e < D; ++e) Wf[D + 1] += 0.25 * P.dt * Wf[1 + e] * P.accel[e];
    }
    return primitives(P, D, Wf);
}

// The face's coefficients and flux moments from its sums S and the separable
// discrete moments of its Maxwellian, M[k][p] = sum_m w_m xi_m^p E_k(m).
template <int D>
__device__ __forceinline__ void face_finish(const Problem& P, int dn, unsigned f, const double (&S)[2 * D + 3],
                                            const Prim& q, const double (&M)[D][5]) {
    const long long NE = P.NE;
    const double beta = 0.25 * P.dt * q.inv_tau_g;
    const double betab = beta * P.Pr;
    const double eta = beta * (P.Pr - 1.0);
    const double A = maxwell_prefactor(D, q.rho, q.RT);
    const double inv2RT = 0.5 / q.RT;
    const double hu2 = 0.5 * (q.u[0] * q.u[0] + q.u[1] * q.u[1] + q.u[2] * q.u[2]);
    const double cRT2 = 0.5 * P.c_int * q.RT;
    double* const Go = P.G + (long long)dn * (D + 2) * NE + f;
    // one body per normal, so every index of M and S is a constant
#pragma unroll
    for (int d = 0; d < D; ++d) {
        if (d != dn) continue;
        auto prod0 = [&](int skip1, int skip2) __attribute__((always_inline)) {
            double p = 1.0;
#pragma unroll
            for (int k = 0; k < D; ++k)
                if (k != skip1 && k != skip2) p *= M[k][0];
            return p;
        };
        // equilibrium flux moments through a face with normal d
        double E1 = A * M[d][1] * prod0(d, -1);
        double E2[D];
#pragma unroll
        for (int e = 0; e < D; ++e)
            E2[e] = e == d ? A * M[d][2] * prod0(d, -1) : A * M[d][1] * M[e][1] * prod0(d, e);
        double X3 = M[d][3] * prod0(d, -1);
#pragma unroll
        for (int e = 0; e < D; ++e)
            if (e != d) X3 += M[d][1] * M[e][2] * prod0(d, e);
        X3 *= A;
        double E3 = 0.5 * X3 + cRT2 * E1;
        double EZ = -hu2 * E1;
#pragma unroll
        for (int e = 0; e < D; ++e) EZ += q.u[e] * E2[e];

        // phi at the face is affine in phi_bar (inversion of eq. phibar), so
        // the flux moments follow from the velocity sums of phi_bar and the
        // equilibrium moments above.
        const double ig = 1.0 / (1.0 + beta), ib = 1.0 / (1.0 + betab);
        double Gm = (S[1 + d] + beta * E1) * ig;
        double Gp[D];
#pragma unroll
        for (int e = 0; e < D; ++e) Gp[e] = (S[D + 2 + e] + beta * E2[e]) * ig;
        double accE = 0.0;
        if (P.has_accel) {
            // The acceleration's (h/2) S terms at the face (eqs. gsource,
            // bsource with the velocity derivative on the equilibrium) enter
            // g_f as ig c (a.xi - a.u) g_eq and b_f as ib [(dt/4) a.xi (g_f -
            // g_eq) + c (a.xi - a.u) b_eq], c = (h/2)/(R T); their flux
            // moments need third and fourth separable moments of the face
            // Maxwellian.
            auto mom = [&](const int (&p)[3]) __attribute__((always_inline)) {
                double r = A * M[0][p[0]];
#pragma unroll
                for (int k = 1; k < D; ++k) r *= M[k][p[k]];
                return r;
            };
            const double c = 0.5 * P.dt * inv2RT;
            double au = 0.0, aE2 = 0.0;
#pragma unroll
            for (int k = 0; k < D; ++k) {
                au += P.accel[k] * q.u[k];
                aE2 += P.accel[k] * E2[k];
            }
            Gm += ig * c * (aE2 - au * E1);
#pragma unroll
            for (int e = 0; e < D; ++e) {
                double t3 = 0.0;  // sum_k a_k sum_i w_i xi_d xi_e xi_k g_eq
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    int p[3] = {0, 0, 0};
                    p[d] += 1;
                    p[e] += 1;
                    p[k] += 1;
                    t3 += P.accel[k] * mom(p);
                }
                Gp[e] += ig * c * (t3 - au * E2[e]);
            }
            double aB2 = 0.0, aG = 0.0;  // sum_k a_k sum_i w_i xi_d xi_k b_eq; sum_k a_k (G_k - E2_k)
#pragma unroll
            for (int k = 0; k < D; ++k) {
                double q4 = 0.0;
#pragma unroll
                for (int m = 0; m < D; ++m) {
                    int p[3] = {0, 0, 0};
                    p[d] += 1;
                    p[k] += 1;
                    p[m] += 2;
                    q4 += mom(p);
                }
                aB2 += P.accel[k] * (0.5 * q4 + cRT2 * E2[k]);
                aG += P.accel[k] * (Gp[k] - E2[k]);
            }
            accE = 0.25 * P.dt * aG + c * (aB2 - au * E3);
        }
        double ZG = -hu2 * Gm;
#pragma unroll
        for (int e = 0; e < D; ++e) ZG += q.u[e] * Gp[e];
        double Ge = (S[2 * D + 2] + betab * E3 + eta * (ZG - EZ) + accE) * ib;

        Go[0] = Gm;
#pragma unroll
        for (int e = 0; e < D; ++e) Go[(long long)(1 + e) * NE] = Gp[e];
        Go[(long long)(D + 1) * NE] = Ge;
        double* F = P.FP + (long long)d * NFP * NE + f;
        F[PF_A * NE] = A;
        F[PF_INV2RT * NE] = inv2RT;
        F[PF_CRT2 * NE] = cRT2;
        F[PF_IG * NE] = ig;
        F[PF_IB * NE] = ib;
        F[PF_EB * NE] = eta * ib;
        F[PF_HU2 * NE] = hu2;
#pragma unroll
        for (int e = 0; e < 3; ++e) F[(PF_U0 + e) * NE] = q.u[e];
    }
}

// One thread per face: t counts (normal, face).
template <int D>
__device__ __forceinline__ void face_close_one(const Problem& P, long long t) {
    const unsigned NE = (unsigned)P.NE;
    if (t >= (long long)NE * D) return;
    const int d = (int)(t / NE);
    const unsigned f = (unsigned)(t - (long long)d * NE);
    if (!face_in_grid<D>(P, d, f)) return;
    constexpr int NS = 2 * D + 3;
    double S[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) S[j] = 0.0;
#pragma unroll 2
    for (int s = 0; s < P.nslices; ++s) {
        const double* in = P.FS + ((long long)(s * D + d) * NS) * NE + f;
#pragma unroll
        for (int j = 0; j < NS; ++j) S[j] += in[(long long)j * NE];
    }
    const Prim q = face_primitives<D>(P, S);
    if (q.bad) {
        raise_error(P.err);
        return;
    }
    const double inv2RT = 0.5 / q.RT;
    double M[D][5];
    int off = 0;
#pragma unroll
    for (int k = 0; k < D; ++k) {
#pragma unroll
        for (int p = 0; p < 5; ++p) M[k][p] = 0.0;
#pragma unroll 4
        for (int m = 0; m < P.nv[k]; ++m) {
            double x = P.axis_xi[off + m];
            double e = P.axis_w[off + m] * exp(-(x - q.u[k]) * (x - q.u[k]) * inv2RT);
            M[k][0] += e;
            M[k][1] += e * x;
            M[k][2] += e * x * x;
            M[k][3] += e * x * x * x;
            M[k][4] += e * x * x * x * x;
        }
        off += P.nv[k];
    }
    face_finish<D>(P, d, f, S, q, M);
}

// L neighbouring threads per face.  What is long in a face's closure is the
// exponential per node of each velocity axis and the sums over nodes and over
// velocity slices.  The threads of the group share the exponentials, a chunk
// of nodes at a time, through LDS; then each of its first 5D threads runs one
// moment's sum over the chunk, and before that each of the first 2D+3 one
// velocity sum over the slices.  Every sum is added up in the order of the
// one-thread form, so the group size never changes a result.  With one thread
// per face a step of the 128 x 16385 sine wave spent 2.86 ms of its 3.31 ms in
// this closure, on 1/500 of the device's threads.
// The sums are what is left then, one dependent FMA per node: their operands
// are read 16 nodes ahead, two per LDS access, so an axis is padded to blocks
// of 16 with nodes that add exact zeros.
constexpr int CLOSE_BLOCK = 16;
template <int L>
struct CloseShared {
    static constexpr int NF = WG / L;     // faces per workgroup
    static constexpr int C = 2 * L;       // nodes of a chunk
    static constexpr int ROW = C + 2;     // rows 16 bytes past a multiple of the banks
    double t[NF][5][ROW];                 // w e, w e x, w e x^2, w e x^3, x
    double s[NF][16];                     // velocity sums, then moments
    double one[CLOSE_BLOCK];
};
constexpr int CLOSE_LDS_DOUBLES = 5 * (2 * WG + 2 * WG / 16) + WG + CLOSE_BLOCK;  // the largest is at L = 16
template <int D, int L>
__device__ __forceinline__ void face_close_group(const Problem& P, long long t, double* lds) {
    constexpr int NS = 2 * D + 3;
    using Sh = CloseShared<L>;
    static_assert(NS <= 16 && 5 * D <= 16 && L >= 16, "a group runs its sums one per thread");
    static_assert(sizeof(Sh) <= CLOSE_LDS_DOUBLES * sizeof(double), "closure LDS");
    static_assert(Sh::C % CLOSE_BLOCK == 0, "chunks of whole blocks");
    Sh& sm = *reinterpret_cast<Sh*>(lds);
    const unsigned NE = (unsigned)P.NE;
    const long long idx = t / L;  // face counted over the normals
    const int fi = (int)threadIdx.x / L, lane = (int)threadIdx.x % L;
    // every thread takes part in the barriers; a group without a face works
    // on face 0 and writes nothing
    bool valid = idx < (long long)NE * D;
    const int d = valid ? (int)(idx / NE) : 0;
    const unsigned f = valid ? (unsigned)(idx - (long long)d * NE) : 0;
    valid = valid && face_in_grid<D>(P, d, f);

    // nodes of the axes, each padded to whole blocks, one axis after another;
    // a padding node has weight 0 at x = 0
    auto padded = [](int n) { return (n + CLOSE_BLOCK - 1) / CLOSE_BLOCK * CLOSE_BLOCK; };
    const int e1 = padded(P.nv[0]), e2 = e1 + (D >= 2 ? padded(P.nv[1]) : 0), e3 = e2 + (D >= 3 ? padded(P.nv[2]) : 0);
    double nx[2], nw[2];  // this thread's nodes of the next chunk
    int na[2];            // and their axes (-1: padding)
    const int v0n = P.nv[0], v1n = P.nv[1], v2n = P.nv[2];
    auto load_nodes = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int v = c0 + lane + j * L;
            // position on its axis, the axis' length and its place in the tables
            int ax = 0, m = v, n = v0n, at = 0;
            if (D >= 2 && v >= e1) ax = 1, m = v - e1, n = v1n, at = v0n;
            if (D >= 3 && v >= e2) ax = 2, m = v - e2, n = v2n, at = v0n + v1n;
            const bool in = m < n;
            const int i = in ? at + m : 0;
            na[j] = in ? ax : -1;
            nx[j] = P.axis_xi[i];
            nw[j] = P.axis_w[i];
        }
    };
    load_nodes(0);

    // velocity sums over the slices: the group's threads fetch as many slices
    // as fit the LDS at once, then each of the first NS adds its column up
    if (threadIdx.x < CLOSE_BLOCK) sm.one[threadIdx.x] = 1.0;
    {
        constexpr int NR = 8;             // loads in flight per thread
        constexpr int SC = NR * L / NS;   // slices at once
        static_assert(SC * NS <= 5 * Sh::ROW, "slices of a pass fit the group's LDS");
        double* const part = &sm.t[fi][0][0];
        const double* const in = P.FS + (long long)d * NS * NE + f;
        double a = 0.0;
        for (int s0 = 0; s0 < P.nslices; s0 += SC) {
            const int ns = P.nslices - s0 < SC ? P.nslices - s0 : SC;
            double r[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                // past the pass' last value: reload the first, not stored
                const int i = lane + k * L < ns * NS ? lane + k * L : 0;
                const int s = i / NS, j = i - s * NS;
                r[k] = in[((long long)(s0 + s) * D * NS + j) * NE];
            }
#pragma unroll
            for (int k = 0; k < NR; ++k)
                if (lane + k * L < ns * NS) part[lane + k * L] = r[k];
            __syncthreads();
            if (lane < NS) {
#pragma unroll 8
                for (int s = 0; s < ns; ++s) a += part[s * NS + lane];
            }
            __syncthreads();
        }
        if (lane < NS) sm.s[fi][lane] = a;
    }
    __syncthreads();
    double S[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) S[j] = sm.s[fi][j];
    const Prim q = face_primitives<D>(P, S);
    if (valid && q.bad) {
        if (lane == 0) raise_error(P.err);
        valid = false;
    }
    const double inv2RT = 0.5 / q.RT;
    // this thread's sum: moment p of axis k, over padded nodes [a0, a1)
    const int k = lane / 5, p = lane % 5;
    const int a0 = k == 0 ? 0 : (k == 1 ? e1 : e2);
    const int a1 = lane >= 5 * D ? a0 : (k == 0 ? e1 : (k == 1 ? e2 : e3));
    const int row = p == 0 ? 0 : p - 1;
    // second factors: x, for p = 0 ones (M + e, exactly)
    const double* const xs = p == 0 ? sm.one : sm.t[fi][4];
    const int xstep = p == 0 ? 0 : 1;
    double M = 0.0;
    for (int c0 = 0; c0 < e3; c0 += Sh::C) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int o = lane + j * L;
            const double uk = D == 1 || na[j] <= 0 ? q.u[0] : (D == 2 || na[j] == 1 ? q.u[1] : q.u[2]);
            double x = nx[j];
            double e = nw[j] * exp(-(x - uk) * (x - uk) * inv2RT);
            if (na[j] < 0) x = e = 0.0;
            sm.t[fi][0][o] = e;
            sm.t[fi][1][o] = e * x;
            sm.t[fi][2][o] = e * x * x;
            sm.t[fi][3][o] = e * x * x * x;
            sm.t[fi][4][o] = x;
        }
        load_nodes(c0 + Sh::C);  // in flight behind this chunk's sums
        __syncthreads();
        const int m0 = (a0 > c0 ? a0 : c0) - c0, m1 = (a1 < c0 + Sh::C ? a1 : c0 + Sh::C) - c0;
        if (m0 < m1) {
            double A[2][CLOSE_BLOCK], X[2][CLOSE_BLOCK];
            auto load = [&](int m, int h) __attribute__((always_inline)) {
                const double2* a = reinterpret_cast<const double2*>(&sm.t[fi][row][m]);
                const double2* x = reinterpret_cast<const double2*>(xs + xstep * m);
#pragma unroll
                for (int j = 0; j < CLOSE_BLOCK / 2; ++j) {
                    const double2 va = a[j], vx = x[j];
                    A[h][2 * j] = va.x;
                    A[h][2 * j + 1] = va.y;
                    X[h][2 * j] = vx.x;
                    X[h][2 * j + 1] = vx.y;
                }
            };
            auto sum = [&](int h) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < CLOSE_BLOCK; ++j) M = fma(A[h][j], X[h][j], M);
            };
            load(m0, 0);
            int m = m0;
            for (; m + CLOSE_BLOCK < m1; m += 2 * CLOSE_BLOCK) {
                load(m + CLOSE_BLOCK, 1);
                sum(0);
                // past the last block: reload it, unused
                load(m + 2 * CLOSE_BLOCK < m1 ? m + 2 * CLOSE_BLOCK : m, 0);
                sum(1);
            }
            if (m < m1) sum(0);
        }
        __syncthreads();
    }
    if (lane < 5 * D) sm.s[fi][lane] = M;
    __syncthreads();
    if (lane != 0 || !valid) return;
    double Mf[D][5];
#pragma unroll
    for (int e = 0; e < D; ++e)
#pragma unroll
        for (int j = 0; j < 5; ++j) Mf[e][j] = sm.s[fi][5 * e + j];
    face_finish<D>(P, d, f, S, q, Mf);
}

// by group size
template <int D, int L>
__device__ __forceinline__ void face_close(const Problem& P, long long t, double* lds) {
    if constexpr (L == 1) face_close_one<D>(P, t);
    else face_close_group<D, L>(P, t, lds);
}
template <int D, bool GROUPS>
__device__ __forceinline__ void face_close_lanes(const Problem& P, long long t, double* lds) {
    if constexpr (!GROUPS) return face_close<D, 1>(P, t, lds);
    switch (P.close_lanes) {  // uniform per problem
    case 1: face_close<D, 1>(P, t, lds); break;
    case 16: face_close<D, 16>(P, t, lds); break;
    case 64: face_close<D, 64>(P, t, lds); break;
    default: face_close<D, 256>(P, t, lds); break;
    }
}

// per-problem thread ranges of the batched per-face launch
__device__ __forceinline__ int find_problem(const long long* offsets, int nprob, long long g) {
    int lo = 0, hi = nprob - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) / 2;
        if (offsets[mid] <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

}  // namespace cdg
