// wg.hip -- workgroup tiles with an operation list read at run time: the
// interpreted form of the compiled workgroup passes.  Compiled once per
// direction: -DDQ_WG_ADJ selects the adjoint passes (else the forward ones).
// complex64 only.
//
// A workgroup of four waves owns 2^(6+R+2) amplitudes in registers.  The
// host orders a pass's gates into layouts of the tile (which tile bits are
// lane, register and wave bits) in which the bits that gates exchange are
// register bits, so no operation moves data across lanes; between layouts
// the tile goes through LDS.  Gates of one kind on different register bits
// form one block, and a run of one-qubit diagonal gates anywhere in the tile
// one product diagonal, so that the cost of decoding an operation (scalar
// loads, branches) is paid once per block.  Both matter because these passes
// are bound by instruction issue, not by memory: the one-wave interpreter
// spends about 200 instructions on a one-qubit gate whose arithmetic takes
// 128, and 300 per tile outside its gates.  Two workgroups fit a compute unit
// (64 KiB of exchange buffer and 16 KiB of gradient sums in an adjoint pass).
// Gradient step, one-wave passes -> these: 64 circuits of 12 to 22 qubits
// 26.1 -> 18.0 ms, 12 qubits and 64 samples 368 -> 291 and, with the heads of
// the entries in lanes (WgHeads), 276 us; two layers of CZ or RZZ gates between
// each wire and the next six, 16 qubits, forward 116 and 167 us in one-wave
// passes, 140 and 204 without those heads, 127 and 181 with them.
#include "dq_internal.h"

#include <type_traits>
#include <utility>

namespace dq {
namespace {

constexpr int WB = WG_WAVE_BITS;

__device__ __forceinline__ int rl(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
// one uniform field of a table in the constant address space
__device__ __forceinline__ int fld(cptr<WgOp> o, int k) { return o->a[k]; }
// The first words of the operations, lane l holding those of operation l of
// its group of 64, and in passes with two-qubit diagonal gates (diags) their
// matrices' diagonals: read by scalar loads, an entry and then its matrix are
// two dependent misses of the scalar cache, which nothing hides when few
// workgroups run.
struct WgHead {
    int kind, a0, a1, a2;
};
struct WgHeads {
    WgHead mine;
    float d[8];
    int group = -1;
    __device__ __forceinline__ WgHead of(const WgOp *ops, int nops, int k, const cx<float> *mats, bool diags, int lane) {
        if ((k >> 6) != group) {
            group = k >> 6;
            const int l = (group << 6) + lane;
            const WgOp *o = ops + (l < nops ? l : nops - 1);
            mine = WgHead{o->kind, o->a[0], o->a[1], o->a[2]};
            if (diags) {
                const cx<float> *m = mats + (mine.kind == WG_2QDIAG ? mine.a2 : 0);
                const int step = mine.kind == WG_2QDIAG ? 5 : 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const cx<float> e = m[i * step];
                    d[2 * i] = e.x;
                    d[2 * i + 1] = e.y;
                }
            }
        }
        const int l = k & 63;
        return WgHead{rl(mine.kind, l), rl(mine.a0, l), rl(mine.a1, l), rl(mine.a2, l)};
    }
    __device__ __forceinline__ cx<float> diag(int k, int i) const {
        return cx<float>{__int_as_float(rl(__float_as_int(d[2 * i]), k & 63)), __int_as_float(rl(__float_as_int(d[2 * i + 1]), k & 63))};
    }
};
// static choice by a uniform index: binary, a chain of comparisons costs up to ten
template <int LO, int HI, typename F> __device__ __forceinline__ void pick(int i, F &&f) {
    if constexpr (HI - LO == 1) {
        f(std::integral_constant<int, LO>{});
    } else {
        constexpr int MID = (LO + HI) / 2;
        if (i < MID) pick<LO, MID>(i, f);
        else pick<MID, HI>(i, f);
    }
}
// register bits (a, b), a < b, of pair b (b - 1) / 2 + a
constexpr int pair_hi(int p) { int b = 1; while (b * (b + 1) / 2 <= p) ++b; return b; }
constexpr int pair_lo(int p) { return p - pair_hi(p) * (pair_hi(p) - 1) / 2; }

__device__ __forceinline__ int64_t wg_base(int64_t t, int T, const int32_t *tb) {
    int64_t base = t << 3;
    for (int k = 0; k < T - 3; ++k) base = insert_zero(base, tb[k]);
    return base;
}
__device__ __forceinline__ int64_t wg_lane_off(int lane, const int32_t *phys) {
    int64_t o = 0;
#pragma unroll
    for (int p = 0; p < 6; ++p) o += int64_t((lane >> p) & 1) << phys[p];
    return o;
}
template <int R> __device__ __forceinline__ int64_t wg_wave_off(int wave, const int32_t *phys) {
    int64_t o = 0;
#pragma unroll
    for (int p = 0; p < WB; ++p) o += int64_t((wave >> p) & 1) << phys[6 + R + p];
    return o;
}
template <int R> __device__ __forceinline__ int64_t wg_reg_off(int i, const int32_t *phys) {
    int64_t o = 0;
#pragma unroll
    for (int p = 0; p < R; ++p)
        if ((i >> p) & 1) o += int64_t(1) << phys[6 + p];
    return o;
}

// Layout exchange: real and imaginary parts of every state at once, so that
// an element's index is formed once (one XOR with a uniform mask per
// register; this lane's part comes from a table) and two barriers do.
template <typename T, int NS, int R>
__device__ __forceinline__ void wg_xchg(cx<T> (&v)[NS][1 << R], char *buf, const WgX *xs, int wave, int lane) {
    constexpr int NR = 1 << R, TB = 6 + R + WB;
    const cptr<WgX> x = to_const(xs);
    int wa = xs->lw[lane], ra = xs->lr[lane];
    int ww = 0, rw = 0;
#pragma unroll
    for (int k = 0; k < WB; ++k) {
        ww ^= ((wave >> k) & 1) ? x->w[6 + R + k] : 0;
        rw ^= ((wave >> k) & 1) ? x->r[6 + R + k] : 0;
    }
    int mw[NR], mr[NR];   // uniform
    mw[0] = ww;
    mr[0] = rw;
    static_for<1, NR>([&](auto ic) {
        constexpr int i = decltype(ic)::value, k = 31 - __builtin_clz(i);
        mw[i] = mw[i ^ (1 << k)] ^ x->w[6 + k];
        mr[i] = mr[i ^ (1 << k)] ^ x->r[6 + k];
    });
    lds_barrier();   // earlier reads of the buffer are done
    DQ_SF(NR, {
        T *p = (T *)(buf + (wa ^ mw[i]));
        DQ_NS({
            p[(2 * s_) << TB] = v[s_][i].x;
            p[(2 * s_ + 1) << TB] = v[s_][i].y;
        });
    });
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
    DQ_SF(NR, {
        const T *p = (const T *)(buf + (ra ^ mr[i]));
        DQ_NS({ v[s_][i] = cx<T>{p[(2 * s_) << TB], p[(2 * s_ + 1) << TB]}; });
    });
    __builtin_amdgcn_sched_barrier(0);
}

// In-place arithmetic.  Every operation sits between run-time branches at
// which the tile's values must be in the same registers whichever way was
// taken; left to itself the compiler writes results to fresh registers and
// copies the whole tile back at the joins (64 moves beside the 128 multiply-
// adds of a gate on two states).  Results that overwrite an operand avoid it.
//   a = m a + t (m uniform), the same with m per lane
__device__ __forceinline__ void fma_in(float &a, float m, float t) { asm("v_fma_f32 %0, %1, %0, %2" : "+v"(a) : "s"(m), "v"(t)); }
__device__ __forceinline__ void fma_lane(float &a, float m, float t) { asm("v_fma_f32 %0, %1, %0, %2" : "+v"(a) : "v"(m), "v"(t)); }
// flips the signs of the lanes whose mask is the sign bit (else 0)
__device__ __forceinline__ void flip_in(float &a, int mask) { asm("v_xor_b32 %0, %1, %0" : "+v"(a) : "v"(mask)); }
__device__ __forceinline__ void swap_in(float &a, float &b) { asm volatile("v_swap_b32 %0, %1" : "+v"(a), "+v"(b)); }

// the register forms of tile_dev.h (same operations, same rounding), in place
template <typename T, int NS, int NR, int K>
__device__ __forceinline__ void wg_real(cx<T> (&v)[NS][NR], T m00, T m01, T m10, T m11) {
    DQ_SF(NR / 2, {
        constexpr int i0 = Pair<K>::lo(i), i1 = Pair<K>::hi(i);
        DQ_NS({
            const T tx = m01 * v[s_][i1].x, ty = m01 * v[s_][i1].y, ux = m10 * v[s_][i0].x, uy = m10 * v[s_][i0].y;
            fma_in(v[s_][i0].x, m00, tx);
            fma_in(v[s_][i0].y, m00, ty);
            fma_in(v[s_][i1].x, m11, ux);
            fma_in(v[s_][i1].y, m11, uy);
        });
    });
}
template <typename T, int NS, int NR, int K>
__device__ __forceinline__ void wg_rx(cx<T> (&v)[NS][NR], T c, T s) {
    DQ_SF(NR / 2, {
        constexpr int i0 = Pair<K>::lo(i), i1 = Pair<K>::hi(i);
        DQ_NS({
            const T tx = -s * v[s_][i1].y, ty = s * v[s_][i1].x, ux = -s * v[s_][i0].y, uy = s * v[s_][i0].x;
            fma_in(v[s_][i0].x, c, tx);
            fma_in(v[s_][i0].y, c, ty);
            fma_in(v[s_][i1].x, c, ux);
            fma_in(v[s_][i1].y, c, uy);
        });
    });
}
template <typename T, int NS, int NR, int K>
__device__ __forceinline__ void wg_1q(cx<T> (&v)[NS][NR], cx<T> m00, cx<T> m01, cx<T> m10, cx<T> m11) {
    DQ_SF(NR / 2, {
        constexpr int i0 = Pair<K>::lo(i), i1 = Pair<K>::hi(i);
        DQ_NS({
            const cx<T> a0 = v[s_][i0], a1 = v[s_][i1], t = cmul(m01, a1), u = cmul(m10, a0);
            const T px = fm(-m00.y, a0.y, t.x), py = fm(m00.y, a0.x, t.y);
            const T qx = fm(-m11.y, a1.y, u.x), qy = fm(m11.y, a1.x, u.y);
            fma_in(v[s_][i0].x, m00.x, px);
            fma_in(v[s_][i0].y, m00.x, py);
            fma_in(v[s_][i1].x, m11.x, qx);
            fma_in(v[s_][i1].y, m11.x, qy);
        });
    });
}
// a = f a, f per lane
template <typename T> __device__ __forceinline__ void mul_lane(cx<T> &a, cx<T> f) {
    const T tx = -f.y * a.y, ty = f.y * a.x;
    fma_lane(a.x, f.x, tx);
    fma_lane(a.y, f.x, ty);
}

// exactly 1 (of a uniform value: scalar compares)
__device__ __forceinline__ bool is_one(cx<float> f) { return __float_as_int(f.x) == 0x3f800000 && (__float_as_int(f.y) << 1) == 0; }

__device__ __forceinline__ double rl_f64(float x, int l) { return (double)__int_as_float(rl(__float_as_int(x), l)); }

// A run of one-qubit diagonal gates at any positions as one product diagonal:
// lane j reads gate j, and the gates are taken in order by reading its
// registers.  The lane's factor and the ratio of every register bit are
// formed in float64 and rounded once; an amplitude takes the factor and the
// ratios of its set bits (the compiled passes tabulate the first three
// ratios' products: here that table would not fit beside the tile).
template <typename T, int NS, int R, int... KS>
__device__ __forceinline__ void wg_diag(cx<T> (&v)[NS][1 << R], std::integer_sequence<int, KS...>, const WgDiag *run,
                                        int count, bool grads, const cx<T> *m, int pos, int lane, int wave, double *acc) {
    constexpr int NR = 1 << R;
    using V = cx<T>;
    WgDiag e{0, 0, -1, 0};
    if (lane < count) e = run[lane];
    const V e0 = m[e.slot], e1 = m[e.slot + 3];
    T sa = 0, sk[R > 0 ? R : 1] = {};
    if constexpr (NS == 2) {
        if (grads) run_sums<T, V, NR, KS...>(v[0], v[1], sa, sk);
    }
    C128 fl{1.0, 0.0}, r[R > 0 ? R : 1];
#pragma unroll
    for (int k = 0; k < R; ++k) r[k] = C128{1.0, 0.0};
    unsigned used = 0;   // register bits with a gate
    for (int j = 0; j < count; ++j) {
        const int q = rl(e.q, j);
        const C128 d0{rl_f64(e0.x, j), rl_f64(e0.y, j)}, d1{rl_f64(e1.x, j), rl_f64(e1.y, j)};
        T term = ((pos >> q) & 1) ? -sa : sa;
        if (q >= 6 && q < 6 + R) {
            fl = cmul(fl, d0);
            used |= 1u << (q - 6);
            const C128 ratio = cmul(d1, cconj(d0));
            static_for<0, R>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                if (q == 6 + k) {
                    r[k] = cmul(r[k], ratio);
                    term = sk[k];
                }
            });
        } else {
            fl = cmul(fl, csel(((pos >> q) & 1) != 0, d1, d0));
        }
        if constexpr (NS == 2) {
            const int ls = rl(e.lslot, j);
            if (ls >= 0) wide_acc<WB>(acc, ls, lane, wave, (double)term);
        }
    }
    const V f = narrow<T>(fl);
    DQ_SF(NR, { DQ_NS({ mul_lane(v[s_][i], f); }); });
    static_for<0, R>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if ((used >> k) & 1) {
            const V rk = narrow<T>(r[k]);
            DQ_SF(NR, {
                if constexpr ((i >> k) & 1) { DQ_NS({ mul_lane(v[s_][i], rk); }); }
            });
        }
    });
}

template <typename T, int NS, int R>
__device__ __forceinline__ void wg_ops(cx<T> (&v)[NS][1 << R], cptr<WgOp> ops, int nops, const WgDiag *diag,
                                       const WgX *xs, const cx<T> *mats, bool diags, char *buf, double *acc, int pos, int lane,
                                       int wave) {
    using V = cx<T>;
    constexpr int NR = 1 << R;
    const cptr<V> m = to_const(mats);
    auto isreg = [](int q) { return q >= 6 && q < 6 + R; };
    WgHeads heads;
    for (int k = 0; k < nops; ++k) {
        const cptr<WgOp> o = ops + k;
        const WgHead h = heads.of((const WgOp *)ops, nops, k, mats, diags, lane);
        switch (h.kind) {
        case WG_REAL: {   // one real 2x2 (RY, H, X, Z) on each register bit of the block
            T c[R > 0 ? R : 1][4];
#pragma unroll
            for (int b = 0; b < R; ++b) {
                const int sl = fld(o, 2 * b) < 0 ? 0 : fld(o, 2 * b);
                c[b][0] = m[sl].x;
                c[b][1] = m[sl + 1].x;
                c[b][2] = m[sl + 2].x;
                c[b][3] = m[sl + 3].x;
            }
            static_for<0, R>([&](auto bc) {
                constexpr int b = decltype(bc)::value;
                if (fld(o, 2 * b) >= 0) {
                    if constexpr (NS == 2) {
                        const int ls = fld(o, 2 * b + 1);
                        if (ls >= 0) wide_acc<WB>(acc, ls, lane, wave, (double)reg_xy_sum<T, V, NR, b>(v[0], v[1], true));
                    }
                    wg_real<T, NS, NR, b>(v, c[b][0], c[b][1], c[b][2], c[b][3]);
                }
            });
            break;
        }
        case WG_RX: {
            T c[R > 0 ? R : 1][2];
#pragma unroll
            for (int b = 0; b < R; ++b) {
                const int sl = fld(o, 2 * b) < 0 ? 0 : fld(o, 2 * b);
                c[b][0] = m[sl].x;
                c[b][1] = m[sl + 1].y;
            }
            static_for<0, R>([&](auto bc) {
                constexpr int b = decltype(bc)::value;
                if (fld(o, 2 * b) >= 0) {
                    if constexpr (NS == 2) {
                        const int ls = fld(o, 2 * b + 1);
                        if (ls >= 0) wide_acc<WB>(acc, ls, lane, wave, (double)reg_xy_sum<T, V, NR, b>(v[0], v[1], false));
                    }
                    wg_rx<T, NS, NR, b>(v, c[b][0], c[b][1]);
                }
            });
            break;
        }
        case WG_1Q:   // dense 2x2 (no generator: differentiable gates are RX, RY and diagonal ones)
            static_for<0, R>([&](auto bc) {
                constexpr int b = decltype(bc)::value;
                const int sl = fld(o, 2 * b);
                if (sl >= 0) wg_1q<T, NS, NR, b>(v, ldc(m, sl), ldc(m, sl + 1), ldc(m, sl + 2), ldc(m, sl + 3));
            });
            break;
        case WG_DIAG:
            wg_diag<T, NS, R>(v, std::make_integer_sequence<int, R>{}, diag + h.a0, h.a1, h.a2 != 0, mats,
                              pos, lane, wave, acc);
            break;
        case WG_CNOT: {   // control a[0] anywhere, target register a[1]
            // swaps under the control's branch: in the lanes whose lane or
            // wave bit is set, or of the register pairs whose bit is set
            const int qc = h.a0, kt = h.a1;
            const bool rc = isreg(qc), lc = (pos >> qc) & 1;
            static_for<0, R>([&](auto bc) {
                constexpr int b = decltype(bc)::value;
                if (kt == b) {
                    static_for<0, R>([&](auto cc) {
                        constexpr int c = decltype(cc)::value;
                        if (c != b && qc == 6 + c) {
                            DQ_SF(NR / 2, {
                                constexpr int i0 = Pair<b>::lo(i), i1 = Pair<b>::hi(i);
                                if constexpr ((i0 >> c) & 1) {
                                    DQ_NS({
                                        swap_in(v[s_][i0].x, v[s_][i1].x);
                                        swap_in(v[s_][i0].y, v[s_][i1].y);
                                    });
                                }
                            });
                        }
                    });
                    if (!rc && lc) {
                        DQ_SF(NR / 2, {
                            constexpr int i0 = Pair<b>::lo(i), i1 = Pair<b>::hi(i);
                            DQ_NS({
                                swap_in(v[s_][i0].x, v[s_][i1].x);
                                swap_in(v[s_][i0].y, v[s_][i1].y);
                            });
                        });
                    }
                }
            });
            break;
        }
        case WG_CZ: {     // any positions
            // only the amplitudes with both register bits set change (with every
            // amplitude multiplied by its sign, found register by register, 25
            // qubits and two layers of 25 controlled rotations took 2230 us
            // forward, against 1838 in one-wave passes and 1808 now)
            const int q0 = h.a0, q1 = h.a1;
            const bool r0 = isreg(q0), r1 = isreg(q1), p0 = (pos >> q0) & 1, p1 = (pos >> q1) & 1;
            constexpr int SIGN = (int)0x80000000;
            if (!r0 && !r1) {
                const int flip = p0 && p1 ? SIGN : 0;
                DQ_SF(NR, {
                    DQ_NS({
                        flip_in(v[s_][i].x, flip);
                        flip_in(v[s_][i].y, flip);
                    });
                });
            } else if (r0 != r1) {
                const int flip = (r0 ? p1 : p0) ? SIGN : 0, kr = (r0 ? q0 : q1) - 6;
                pick<0, R>(kr, [&](auto kc) {
                    constexpr int k = decltype(kc)::value;
                    DQ_SF(NR, {
                        if constexpr ((i >> k) & 1) {
                            DQ_NS({
                                flip_in(v[s_][i].x, flip);
                                flip_in(v[s_][i].y, flip);
                            });
                        }
                    });
                });
            } else {
                const int lo = (q0 < q1 ? q0 : q1) - 6, hi = (q0 < q1 ? q1 : q0) - 6;
                pick<0, R *(R - 1) / 2>(hi * (hi - 1) / 2 + lo, [&](auto pc) {
                    constexpr int a = pair_lo(decltype(pc)::value), b = pair_hi(decltype(pc)::value);
                    DQ_SF(NR, {
                        if constexpr (((i >> a) & 1) && ((i >> b) & 1)) {
                            DQ_NS({
                                flip_in(v[s_][i].x, SIGN);
                                flip_in(v[s_][i].y, SIGN);
                            });
                        }
                    });
                });
            }
            break;
        }
        case WG_2QDIAG: { // diag over (a[0] = msb, a[1]); slot a[2], generator a[3], gradient slot a[4]
            const int q0 = h.a0, q1 = h.a1;
            const bool r0 = isreg(q0), r1 = isreg(q1);
            const bool p0 = (pos >> q0) & 1, p1 = (pos >> q1) & 1;
            const int ls = NS == 2 ? fld(o, 4) : -1;
            const bool zz = fld(o, 3) == GEN_ZZ;   // else |11><11|
            auto term = [&](T s) {
                if constexpr (NS == 2) wide_acc<WB>(acc, ls, lane, wave, (double)s);
            };
            const V d0 = heads.diag(k, 0), d1 = heads.diag(k, 1), d2 = heads.diag(k, 2), d3 = heads.diag(k, 3);
            // the factors by the values of the register bits among the two
            // (a lane or wave bit's value is this lane's)
            // a controlled phase: only the amplitudes with both bits set change
            const bool cp = is_one(d0) && is_one(d1) && is_one(d2);
            const V f00 = csel(!r0 && p0, csel(!r1 && p1, d3, d2), csel(!r1 && p1, d1, d0));
            if (!r0 && !r1) {
                if constexpr (NS == 2)
                    if (ls >= 0) {
                        const T s = all_sum<T, V, NR>(v[0], v[1]);
                        term(zz ? (p0 != p1 ? -s : s) : (p0 && p1 ? s : T(0)));
                    }
                if (!cp || (p0 && p1)) DQ_SF(NR, { DQ_NS({ mul_lane(v[s_][i], f00); }); });
            } else if (r0 != r1) {
                const V f1 = r0 ? csel(p1, d3, d2) : csel(p0, d3, d1);
                const int kr = (r0 ? q0 : q1) - 6;
                const bool p = r0 ? p1 : p0;
                pick<0, R>(kr, [&](auto kc) {
                    constexpr int k = decltype(kc)::value;
                    if constexpr (NS == 2)
                        if (ls >= 0) {
                            if (zz) {
                                const T s = reg_z_sum<T, V, NR, k>(v[0], v[1]);
                                term(p ? -s : s);
                            } else {
                                const T s = reg_set_sum<T, V, NR, k>(v[0], v[1]);
                                term(p ? s : T(0));
                            }
                        }
                    if (!cp) {
                        DQ_SF(NR, {
                            if constexpr (!((i >> k) & 1)) { DQ_NS({ mul_lane(v[s_][i], f00); }); }
                        });
                    }
                    if (!cp || p) {
                        DQ_SF(NR, {
                            if constexpr ((i >> k) & 1) { DQ_NS({ mul_lane(v[s_][i], f1); }); }
                        });
                    }
                });
            } else {
                const int lo = (q0 < q1 ? q0 : q1) - 6, hi = (q0 < q1 ? q1 : q0) - 6;
                const V flo = q0 < q1 ? d2 : d1, fhi = q0 < q1 ? d1 : d2;   // only the lower, only the higher bit set
                pick<0, R *(R - 1) / 2>(hi * (hi - 1) / 2 + lo, [&](auto pc) {
                    constexpr int a = pair_lo(decltype(pc)::value), b = pair_hi(decltype(pc)::value);
                    if constexpr (NS == 2)
                        if (ls >= 0) {
                            if (zz) term(reg_zz_sum<T, V, NR, a, b>(v[0], v[1]));
                            else term(reg_p11_sum<T, V, NR, a, b>(v[0], v[1]));
                        }
                    DQ_SF(NR, {
                        constexpr int x = ((i >> a) & 1) + 2 * ((i >> b) & 1);
                        if constexpr (x == 3) { DQ_NS({ mul_lane(v[s_][i], d3); }); }
                    });
                    if (!cp) {
                        DQ_SF(NR, {
                            constexpr int x = ((i >> a) & 1) + 2 * ((i >> b) & 1);
                            const V f = x == 0 ? d0 : x == 1 ? flo : fhi;
                            if constexpr (x != 3) { DQ_NS({ mul_lane(v[s_][i], f); }); }
                        });
                    }
                });
            }
            break;
        }
        case WG_XCHG:
            wg_xchg<T, NS, R>(v, buf, xs + h.a0, wave, lane);
            break;
        default: break;
        }
    }
}

// One pass over the tiles t0, t0 + step, ... < t1 of one sample.
template <typename T, int NS, int R>
__device__ __forceinline__ void wg_tiles(const WgPass &a, cx<T> *st, cx<T> *lam, const cx<T> *mats, int64_t t0,
                                         int64_t t1, int64_t step, char *buf, double *acc) {
    using V = cx<T>;
    constexpr int NR = 1 << R;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int pos = lane | (wave << (6 + R));
    const int64_t li = wg_lane_off(lane, a.pin), lo = wg_lane_off(lane, a.pout);
    const int64_t wi = wg_wave_off<R>(wave, a.pin), wo = wg_wave_off<R>(wave, a.pout);
    cx<T> *const base_of[2] = {st, lam};
    for (int64_t t = t0; t < t1; t += step) {
        int64_t base = wg_base(t, 6 + R + WB, a.tbits);
        V v[NS][NR];
        DQ_NS({
            const V *p = base_of[s_] + base + wi;
            if (a.nt) {
                DQ_SF(NR, { v[s_][i] = ld_stream(p + wg_reg_off<R>(i, a.pin) + li); });
            } else {
                DQ_SF(NR, { v[s_][i] = (p + wg_reg_off<R>(i, a.pin))[li]; });
            }
        });
        wg_ops<T, NS, R>(v, to_const(a.ops), a.nops, a.diag, a.xs, mats, a.diags != 0, buf, acc, pos, lane, wave);
        asm volatile("" : "+s"(base));
        DQ_NS({
            V *p = base_of[s_] + base + wo;
            if (a.nt) {
                DQ_SF(NR, { st_stream(p + wg_reg_off<R>(i, a.pout) + lo, v[s_][i]); });
            } else {
                DQ_SF(NR, { (p + wg_reg_off<R>(i, a.pout))[lo] = v[s_][i]; });
            }
        });
    }
}

constexpr int BLOCK = 64 << WB;

// a table entry's fields through the constant address space (scalar loads)
__device__ __forceinline__ WgEntry ld_wg_entry(const WgEntry *ents, int e) {
    static_assert(sizeof(WgEntry) % 4 == 0, "copied by words");
    constexpr int N = sizeof(WgEntry) / 4;
    const cptr<int32_t> p = to_const((const int32_t *)(ents + e));
    int32_t w[N];
#pragma unroll
    for (int k = 0; k < N; ++k) w[k] = p[k];
    return __builtin_bit_cast(WgEntry, w);
}
__device__ __forceinline__ int find_wg_entry(const WgEntry *ents, int nent, int64_t u) {
    int lo = 0, hi = nent - 1;
    while (lo < hi) {   // last entry with unit_begin <= u
        const int mid = (lo + hi + 1) >> 1;
        if (to_const(ents)[mid].unit_begin <= u) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

#ifndef DQ_WG_ADJ
template <typename T, int R> constexpr size_t wg_lds() { return 2 * sizeof(T) << (6 + R + WB); }

template <typename T, int R>
__global__ __launch_bounds__(BLOCK, 2) void k_wg_fwd(WgPass a, cx<T> *st, const cx<T> *mats, int64_t mstride, int64_t batch) {
    __shared__ __align__(16) char buf[wg_lds<T, R>()];
    const int ts = a.n - 6 - R - WB;
    const int64_t total = batch << ts, mask = (int64_t(1) << ts) - 1;
    for (int64_t u = blockIdx.x; u < total; u += gridDim.x) {
        const int64_t b = u >> ts, t = u & mask;
        wg_tiles<T, 1, R>(a, st + (b << a.n), nullptr, mats + b * mstride, t, t + 1, 1, buf, nullptr);
    }
}
template <typename T, int R>
__global__ __launch_bounds__(BLOCK, 2) void k_wg_fwd_multi(cx<T> *st, char *ws, const WgEntry *ents, int nent,
                                                           int64_t units) {
    __shared__ __align__(16) char buf[wg_lds<T, R>()];
    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const WgEntry E = ld_wg_entry(ents, find_wg_entry(ents, nent, u));
        const int64_t t = u - E.unit_begin;
        wg_tiles<T, 1, R>(E.pass, st + E.st_off, nullptr, (const cx<T> *)(ws + E.mats_off), t, t + 1, 1, buf, nullptr);
    }
}
#else
// sums a wave's accumulators over the workgroup into the unit's partial row
__device__ __forceinline__ void wg_sums(const WgPass &a, double *row, double *acc) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    lds_barrier();
    for (int s = wave; s < a.nls; s += 1 << WB) {
        double x = lane < (8 << WB) ? acc[(s << (WB + 3)) + lane] : 0.0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
        if (lane == 0) row[a.lsg[s]] = x;
    }
}
template <typename T, int R>
__device__ __forceinline__ void wg_adj_unit(const WgPass &a, cx<T> *st, cx<T> *lam, const cx<T> *mats, int64_t w,
                                            int64_t wps, double *row, char *buf, double *acc) {
    static_assert((8 << WB) <= 64, "at most one accumulator entry per lane of a wave");
    for (int k = threadIdx.x; k < a.nls << (WB + 3); k += BLOCK) acc[k] = 0.0;
    lds_barrier();
    wg_tiles<T, 2, R>(a, st, lam, mats, w, int64_t(1) << (a.n - 6 - R - WB), wps, buf, acc);
    wg_sums(a, row, acc);
}
template <typename T, int R> constexpr size_t wg_lds() { return 4 * sizeof(T) << (6 + R + WB); }

template <typename T, int R>
__global__ __launch_bounds__(BLOCK, 2) void k_wg_adj(WgPass a, cx<T> *st, cx<T> *lam, const cx<T> *mats, int64_t mstride,
                                                     double *partial, int ngrad) {
    __shared__ __align__(16) char buf[wg_lds<T, R>()];
    extern __shared__ double acc[];
    const int64_t b = blockIdx.y, wps = gridDim.x;
    wg_adj_unit<T, R>(a, st + (b << a.n), lam + (b << a.n), mats + b * mstride, blockIdx.x, wps,
                      partial + (b * wps + blockIdx.x) * (int64_t)ngrad, buf, acc);
}
template <typename T, int R>
__global__ __launch_bounds__(BLOCK, 2) void k_wg_adj_multi(cx<T> *st, char *ws, const WgEntry *ents, int nent) {
    __shared__ __align__(16) char buf[wg_lds<T, R>()];
    extern __shared__ double acc[];
    const int64_t u = blockIdx.x;
    const WgEntry E = ld_wg_entry(ents, find_wg_entry(ents, nent, u));
    const int64_t w = u - E.unit_begin;
    wg_adj_unit<T, R>(E.pass, st + E.st_off, (cx<T> *)(ws + E.lam_off), (const cx<T> *)(ws + E.mats_off), w, E.wps,
                      (double *)(ws + E.part_off) + w * (int64_t)E.ngrad, buf, acc);
}
#endif

}  // namespace

using T = float;

#define DQ_WG_1(RN, ...) \
    case RN: { constexpr int RC = RN; __VA_ARGS__; } break;
#ifndef DQ_WG_ADJ
#define DQ_WG_R(R_, ...)                                                                                     \
    switch (R_) {                                                                                            \
        DQ_WG_1(2, __VA_ARGS__) DQ_WG_1(3, __VA_ARGS__) DQ_WG_1(4, __VA_ARGS__) DQ_WG_1(5, __VA_ARGS__)      \
    default: return hipErrorInvalidValue;                                                                    \
    }
hipError_t wg_fwd(const WgPass &a, void *st, const void *mats, int64_t mstride, int64_t batch, hipStream_t s) {
    // two workgroups stay resident per compute unit; four rounds of them
    // even out the end of the pass
    const int64_t tiles = batch << (a.n - 6 - a.R - WB);
    const unsigned g = (unsigned)(tiles < 2048 ? tiles : 2048);
    DQ_WG_R(a.R, hipLaunchKernelGGL((k_wg_fwd<T, RC>), dim3(g), dim3(BLOCK), 0, s, a, (cx<T> *)st, (const cx<T> *)mats,
                                    mstride, batch));
    return hipGetLastError();
}
hipError_t wg_fwd_multi(int R, void *st, void *ws, const WgEntry *e, int32_t n, int64_t units, hipStream_t s) {
    const unsigned g = (unsigned)(units < 16384 ? units : 16384);
    DQ_WG_R(R, hipLaunchKernelGGL((k_wg_fwd_multi<T, RC>), dim3(g), dim3(BLOCK), 0, s, (cx<T> *)st, (char *)ws, e, n, units));
    return hipGetLastError();
}
#else
#define DQ_WG_R(R_, ...)                                                                                     \
    switch (R_) {                                                                                            \
        DQ_WG_1(2, __VA_ARGS__) DQ_WG_1(3, __VA_ARGS__) DQ_WG_1(4, __VA_ARGS__)                              \
    default: return hipErrorInvalidValue;                                                                    \
    }
static size_t acc_bytes(int32_t nls) { return (sizeof(double) << (WB + 3)) * (size_t)(nls > 0 ? nls : 1); }
hipError_t wg_adj(const WgPass &a, void *st, void *lam, const void *mats, int64_t mstride, double *partial,
                         int32_t wps, int32_t ngrad, int64_t batch, hipStream_t s) {
    DQ_WG_R(a.R, hipLaunchKernelGGL((k_wg_adj<T, RC>), dim3((unsigned)wps, (unsigned)batch), dim3(BLOCK), acc_bytes(a.nls), s,
                                    a, (cx<T> *)st, (cx<T> *)lam, (const cx<T> *)mats, mstride, partial, ngrad));
    return hipGetLastError();
}
hipError_t wg_adj_multi(int R, void *st, void *ws, const WgEntry *e, int32_t n, int64_t units, int32_t max_nls,
                               hipStream_t s) {
    DQ_WG_R(R, hipLaunchKernelGGL((k_wg_adj_multi<T, RC>), dim3((unsigned)units), dim3(BLOCK), acc_bytes(max_nls), s,
                                  (cx<T> *)st, (char *)ws, e, n));
    return hipGetLastError();
}
#endif

}  // namespace dq
