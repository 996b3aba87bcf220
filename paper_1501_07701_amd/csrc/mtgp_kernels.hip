// mtgp_kernels.hip -- gfx950 kernels for bulk MTGP32 generation.
//
// One stream per thread group (the paper's per-block generator scope, Sec. 2
// and Sec. 3.2): a group is either one 64-lane wave (several independent
// streams per workgroup, no s_barrier) or a whole workgroup.  The stream's
// N-word state lives in an LDS buffer while it runs (shared memory, Sec. 2)
// and in device memory between launches.
//
// Step structure.  With W = N - pos, the new words x_n .. x_{n+W-1} depend
// only on words older than x_n, so one step produces up to W outputs at once:
// every lane loads its taps for up to K outputs, computes, writes the new
// words to LDS and the tempered outputs to HBM, then the group synchronises
// once.  Steps are rounded down to multiples of 32 words when W >= 64 so that
// the stores of a step cover whole 128-byte lines.  The LDS buffer is linear
// (x_n at a fixed offset from the step's head) so that every tap is an
// immediate offset from one or two per-lane base registers; when the head
// reaches the end of the buffer the last N words are copied to the front.
//
// Jump-ahead.  A work item may start from any state: a long stream is cut
// into segments whose start states jump_block computes from the stream's
// first words (the generator is GF(2)-linear, so the state J outputs ahead
// is a fixed XOR-combination of consecutive words, given by x^(J-1) mod p
// for a polynomial p that annihilates the word sequence).  Each segment
// checks that its final state equals the next segment's jumped start state.
//
// Work is bit-level GF(2) arithmetic: no MFMA.  The bound is HBM write
// bandwidth (4 bytes per output), with VALU and LDS close behind.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <map>
#include <mutex>

#include "mtgp.h"
#include "mtgp_device.h"
#include "mtgp_internal.hpp"

namespace mtgp {

// Batch workspace of mtgp_generate_batch_noalloc: one per GPU, held until
// the process ends.  Host code never passes this name to a kernel (it is a
// host-side stand-in there); it uses the device address that
// scratch_address() looked up on that device.
static __device__ __align__(256) uint8_t scratch[MTGP_NOALLOC_SCRATCH_BYTES];

hipError_t scratch_address(void **out) {
    static std::mutex mu;
    static std::map<int, void *> addr;  // per device
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lk(mu);
    auto it = addr.find(dev);
    if (it == addr.end()) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));  // with `dev` current
        if (e != hipSuccess) return e;
        it = addr.emplace(dev, p).first;
    }
    *out = it->second;
    return hipSuccess;
}

// Pointer into global memory (address space 1), so stores are emitted as
// global_store rather than flat_store.
template <typename T>
using gptr = __attribute__((address_space(1))) T *;

// Pointer into LDS (address space 3).
template <typename T>
using lptr = __attribute__((address_space(3))) T *;

// a ^ b ^ c in one VALU operation (v_bitop3_b32 with truth table 0x96, the
// odd-parity function of its three inputs); hipcc keeps XOR chains as
// two-input operations.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

template <int TPS>
__device__ __forceinline__ void group_sync() {
    if constexpr (TPS == 64) {
        // One wave: LDS operations issue in order, so only the compiler
        // must be kept from moving loads across the step boundary.
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// LDS buffer length (words) for a stream of N words and up to SMAX outputs
// per step, with room for about four steps between compactions.  Several
// waves need at least 2N + SMAX so the compaction copy never overlaps
// itself; a single wave copies overlapping ranges safely and needs only
// N + SMAX.
__host__ __device__ constexpr int buf_words(int N, int SMAX, int TPS) {
    return ((TPS == 64 ? N : 2 * N) + 4 * SMAX + 63) / 64 * 64;
}

// GRP: with room for groups (segment launches of batches that have them; a
// group takes nearly twice the LDS of the other paths, so launches that run
// none keep the smaller block: 16,000 mexp-3217 streams of 3,000 outputs
// 127 us against 167).
template <int N, int TPS, int K, bool GRP = false>
struct Core {
    static constexpr int SMAX = TPS * K;
    static constexpr int BUF = buf_words(N, SMAX, TPS);
    static_assert(BUF >= (TPS == 64 ? N : 2 * N) + SMAX, "compaction would overlap");
    static_assert(N > 64, "the small-step path assumes N > 64");
    // Window path (one wave, W < 64, linear table): a buffer of at least
    // N + WNMAX words, then the recursion and output tables, a 64-word
    // exchange area and the scan matrices.  The per-wave LDS block is the
    // larger of the two layouts; the window buffer takes whatever the
    // wide layout leaves.
    static constexpr int WNMAX = (N - 1) < 64 * WIN_EMAX ? (N - 1) : 64 * WIN_EMAX;
    static constexpr int WTAIL = 32 + 64 + WIN_MAXROUNDS * WIN_MAT_WORDS;
    static constexpr int WLDS = (N + WNMAX + 63) / 64 * 64 + WTAIL;
    // Group path: the members' buffers (eight of a state and two windows, or
    // fewer longer ones), the tables and the scan matrices.
    static constexpr bool GROUPS = GRP;
    static_assert(!GRP || (TPS == 64 && has_groups(N)), "groups: one wave, a short state");
    static constexpr int GTAIL = 32 + GROUP_ROUNDS * WIN_MAT_WORDS;
    static constexpr int GLDS = GROUPS ? 8 * (N + 2 * 64) + GTAIL : 0;
    static constexpr int WIDE_LDS = (BUF + 32) > WLDS ? (BUF + 32) : WLDS;
    static constexpr int LDS_WORDS = WIDE_LDS > GLDS ? WIDE_LDS : GLDS;
    static constexpr int GBUF = LDS_WORDS - GTAIL;
    static constexpr int WBUF = LDS_WORDS - WTAIL;
    static_assert(WBUF >= N + WNMAX, "window buffer too small");

    struct Step {  // per-item values, uniform across the group
        uint32_t pos, sh1, sh2, mask, W;
        uint32_t rb0, rb1, rb2, rb3;  // basis of a linear recursion table
    };

    // x = Y ^ rec[Y & 15]: from LDS, or for a linear table as the XOR of
    // the basis words selected by the low four bits of Y (no LDS round trip
    // on the dependent chain).
    template <bool LIN>
    static __device__ __forceinline__ uint32_t rec(const Step &p, const uint32_t *tbl,
                                                   uint32_t Y) {
        if constexpr (LIN) {
            return rec_reg(p, Y);
        } else {
            return Y ^ tbl[Y & 15u];
        }
    }

    // The linear table's with a bit mask and a three-input operation
    // (0x78: a ^ (b & c)) per basis word.
    static __device__ __forceinline__ uint32_t rec_reg(const Step &p, uint32_t Y) {
        uint32_t a = __builtin_amdgcn_bitop3_b32(Y, (uint32_t)__builtin_amdgcn_sbfe((int)Y, 0, 1),
                                                 p.rb0, 0x78);
        a = __builtin_amdgcn_bitop3_b32(a, (uint32_t)__builtin_amdgcn_sbfe((int)Y, 1, 1), p.rb1,
                                        0x78);
        a = __builtin_amdgcn_bitop3_b32(a, (uint32_t)__builtin_amdgcn_sbfe((int)Y, 2, 1), p.rb2,
                                        0x78);
        return __builtin_amdgcn_bitop3_b32(a, (uint32_t)__builtin_amdgcn_sbfe((int)Y, 3, 1), p.rb3,
                                           0x78);
    }

    template <bool F32>
    static __device__ __forceinline__ uint32_t temper(const uint32_t *tbl, uint32_t x,
                                                      uint32_t hh) {
        uint32_t H = hh ^ (hh >> 16);
        H ^= H >> 8;
        const uint32_t tv = tbl[16 + (H & 15u)];
        if constexpr (F32)
            return __float_as_uint(__uint_as_float((x >> 9) ^ tv) - 1.0f);
        else
            return x ^ tv;
    }

    // Copies the newest N words to the front of the buffer when a step of
    // `reach` words would run past its end (LIM words).  With several waves
    // the source [h-N, h) and destination [0, N) never overlap
    // (h > BUF - SMAX >= 2N); a single wave may copy with overlap, which is
    // safe because its LDS reads and writes execute in instruction order and
    // the copy moves words towards lower addresses.
    // The copy runs in chunks of up to 8 words per lane, all reads of a chunk
    // issued before its writes; a later chunk's sources lie above every
    // earlier chunk's destinations (h > N), so chunking keeps that order.
    template <int LIM = BUF>
    static __device__ __forceinline__ void maybe_compact(uint32_t *buf, uint32_t &h,
                                                         uint32_t reach, uint32_t lane) {
        if (h + reach > (uint32_t)LIM) {
            constexpr int R = (N + TPS - 1) / TPS;
            constexpr int CH = R < 8 ? R : 8;
            const uint32_t *src = buf + (h - N);
#pragma unroll
            for (int j0 = 0; j0 < R; j0 += CH) {
                uint32_t tmp[CH];
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const uint32_t i = lane + (uint32_t)(j0 + j) * TPS;
                    tmp[j] = (j0 + j < R && i < (uint32_t)N) ? src[i] : 0u;
                }
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const uint32_t i = lane + (uint32_t)(j0 + j) * TPS;
                    if (j0 + j < R && i < (uint32_t)N) buf[i] = tmp[j];
                }
            }
            group_sync<TPS>();
            h = N;
        }
    }

    // Steps with W < 64 on one wave: S = W outputs per step, lane l makes
    // x_{h+l}.  Its tap x_{h+l-W} is the word it made in the previous step,
    // so the dependent chain never leaves registers.  The next step's LDS
    // loads are issued right after this step's word is stored, and this
    // step's tempering and output store run while they are in flight.
    template <bool F32, bool LIN>
    static __device__ __forceinline__ void steps_small(const Step &p, uint32_t *__restrict__ buf,
                                                       const uint32_t *__restrict__ tbl,
                                                       gptr<uint32_t> gout, gptr<uint32_t> raw,
                                                       bool want_raw, uint64_t count,
                                                       uint32_t &h, uint64_t &done,
                                                       uint32_t lane) {
        const uint32_t W = p.W;
        maybe_compact(buf, h, 64, lane);
        uint32_t c = buf[h - W + lane];  // in bounds for every lane: h >= N > 64
        uint32_t a = buf[h + lane - N], b = buf[h + lane - N + 1];
        uint32_t hh = buf[h + lane - W - 1];
        while (done < count) {
            const uint64_t rem = count - done;
            const uint32_t S = rem < W ? (uint32_t)rem : W;
            const uint32_t X = (a & p.mask) ^ b;
            const uint32_t x = rec<LIN>(p, tbl, xor3(X, X << p.sh1, c >> p.sh2));
            // lanes >= S write into the next step's slots, which it rewrites
            buf[h + lane] = x;
            const uint32_t hh_cur = hh;
            uint32_t hn = h + S;
            group_sync<TPS>();
            maybe_compact(buf, hn, 64, lane);
            a = buf[hn + lane - N];
            b = buf[hn + lane - N + 1];
            hh = buf[hn + lane - W - 1];
            const uint32_t r = temper<F32>(tbl, x, hh_cur);
            if (lane < S) {
                gout[done + lane] = r;
                if (want_raw) raw[N + done + lane] = x;
            }
            c = x;
            h = hn;
            done += S;
        }
    }

    // y = P v for a 32x32 GF(2) matrix given as 8 nibble tables of 16 words.
    static __device__ __forceinline__ uint32_t mat_apply(const uint32_t *t, uint32_t v) {
        uint32_t y = t[(v & 15u)] ^ t[16 + ((v >> 4) & 15u)];
#pragma unroll
        for (int k = 2; k < 8; k += 2)
            y = xor3(y, t[k * 16 + ((v >> (4 * k)) & 15u)], t[k * 16 + 16 + ((v >> (4 * k + 4)) & 15u)]);
        return y;
    }

    // Windowed steps for W < 64 with a linear recursion table, one wave.
    // A window of wn <= N-1 words only reads words older than its start for
    // x_{n-N} and x_{n-N+1}, so all of them are loaded first.  What remains
    // is the tap chain x_n = G(X_n) ^ M x_{n-W} per residue class n mod W,
    // which is affine: class r is cut into q chunks of E elements (one lane
    // each); every lane runs its chunk from a zero carry, a Hillis-Steele
    // scan with M^(E*2^k) gives each lane its true carry, and the lane
    // reruns its chunk from it.  Tempering and stores then run as one
    // coalesced pass over the window.  E is a compile-time constant so the
    // element loops are straight-line; lanes past the window end compute
    // junk that they write to the exchange area.
    template <bool F32, int E>
    static __device__ __forceinline__ void steps_window_e(const Step &p,
                                                          const uint32_t *__restrict__ prm,
                                                          uint32_t *__restrict__ buf,
                                                          gptr<uint32_t> gout, gptr<uint32_t> raw,
                                                          bool want_raw, uint64_t count,
                                                          uint32_t &h, uint64_t &done,
                                                          uint32_t lane) {
        const uint32_t *tbl = buf + WBUF;
        uint32_t *scr = buf + WBUF + 32;
        uint32_t *mats = scr + 64;
        const uint32_t W = p.W;
        const uint32_t wn = prm[P_WIN_WN], q = prm[P_WIN_Q];
        const uint32_t rounds = prm[P_WIN_ROUNDS];
        for (uint32_t i = lane; i < rounds * WIN_MAT_WORDS; i += 64) mats[i] = prm[P_WIN_MAT + i];
        const uint32_t r = lane / q, sub = lane - (lane / q) * q;
        const bool lane_ok = r < W;
        const uint32_t i0 = sub * (uint32_t)E;
        const uint32_t off0 = r + W * i0;  // the lane's first element in the window
        group_sync<TPS>();
        while (done < count) {
            const uint64_t rem = count - done;
            const uint32_t wc = rem < wn ? (uint32_t)rem : wn;
            maybe_compact<WBUF>(buf, h, wc, lane);
            // this lane's elements: class r, indices i0 .. i0+cnt-1
            const uint32_t lr = (lane_ok && wc > r) ? (wc - 1 - r) / W + 1 : 0u;
            const uint32_t cnt = lr > i0 ? (lr - i0 < (uint32_t)E ? lr - i0 : (uint32_t)E) : 0u;
            uint32_t X[E];
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const uint32_t idx = ((uint32_t)j < cnt) ? h + off0 + W * j - N : h - N;
                const uint32_t a = buf[idx], b = buf[idx + 1];
                const uint32_t x0 = (a & p.mask) ^ b;
                X[j] = x0 ^ (x0 << p.sh1);
            }
            // chunk from a zero carry (the first chunk of a class from its
            // true carry, the class's last word before the window)
            uint32_t c = (sub == 0 && lane_ok) ? buf[h + r - W] : 0u;
            uint32_t v[E];
#pragma unroll
            for (int j = 0; j < E; ++j) {
                c = rec<false>(p, tbl, X[j] ^ (c >> p.sh2));
                v[j] = c;
            }
            if (rounds) {
                // u_s <- u_s ^ M^(E*d) u_{s-d}: true last word of each chunk
                uint32_t u = v[E - 1];
                for (uint32_t k = 0; k < rounds; ++k) {
                    const uint32_t d = 1u << k;
                    scr[lane] = u;
                    group_sync<TPS>();
                    const uint32_t w = scr[sub >= d ? lane - d : lane];
                    group_sync<TPS>();
                    if (sub >= d) u ^= mat_apply(mats + k * WIN_MAT_WORDS, w);
                }
                scr[lane] = u;
                group_sync<TPS>();
                const uint32_t cin = scr[sub > 0 ? lane - 1 : lane];
                group_sync<TPS>();
                if (sub > 0) {
                    c = cin;
#pragma unroll
                    for (int j = 0; j < E; ++j) {
                        c = rec<false>(p, tbl, X[j] ^ (c >> p.sh2));
                        v[j] = c;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const uint32_t dst = ((uint32_t)j < cnt) ? h + off0 + W * j : WBUF + 32 + lane;
                buf[dst] = v[j];
            }
            group_sync<TPS>();
            // tempering and stores, coalesced over the window
            for (uint32_t pp = lane; pp < wc; pp += 64) {
                const uint32_t x = buf[h + pp];
                const uint32_t hh = buf[h + pp - W - 1];
                gout[done + pp] = temper<F32>(tbl, x, hh);
                if (want_raw) raw[N + done + pp] = x;
            }
            group_sync<TPS>();
            h += wc;
            done += wc;
        }
    }

    // The same window for a wave that runs alone or nearly so (plain calls
    // of few streams, prefixes), where the dependent chain and not the work
    // sets the time: the recursion table in registers (48 cycles an element
    // instead of 100), lanes exchange words by shuffles, and tempering keeps
    // four rows' LDS reads in flight.
    template <bool F32, int E>
    static __device__ __forceinline__ void steps_window_lat(const Step &p,
                                                            const uint32_t *__restrict__ prm,
                                                            uint32_t *__restrict__ buf,
                                                            gptr<uint32_t> gout, gptr<uint32_t> raw,
                                                            bool want_raw, uint64_t count,
                                                            uint32_t &h, uint64_t &done,
                                                            uint32_t lane) {
        const uint32_t *tbl = buf + WBUF;
        uint32_t *mats = buf + WBUF + 32 + 64;
        const uint32_t W = p.W;
        const uint32_t wn = prm[P_WIN_WN], q = prm[P_WIN_Q];
        const uint32_t rounds = prm[P_WIN_ROUNDS];
        for (uint32_t i = lane; i < rounds * WIN_MAT_WORDS; i += 64) mats[i] = prm[P_WIN_MAT + i];
        const uint32_t r = lane / q, sub = lane - (lane / q) * q;
        const bool lane_ok = r < W;
        const uint32_t off0 = r + W * (sub * (uint32_t)E);  // the lane's first element
        group_sync<TPS>();
        while (done < count) {
            const uint64_t rem = count - done;
            const uint32_t wc = rem < wn ? (uint32_t)rem : wn;
            maybe_compact<WBUF>(buf, h, wc, lane);
            const uint32_t left = lane_ok && off0 < wc ? wc - off0 : 0u;  // words from off0 on
            uint32_t X[E];
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const uint32_t idx = W * j < left ? h + off0 + W * j - N : h - N;
                const uint32_t x0 = (buf[idx] & p.mask) ^ buf[idx + 1];
                X[j] = x0 ^ (x0 << p.sh1);
            }
            uint32_t c = (sub == 0 && lane_ok) ? buf[h + r - W] : 0u;
            if (rounds) {
                uint32_t u = c;
#pragma unroll
                for (int j = 0; j < E; ++j) u = rec_reg(p, X[j] ^ (u >> p.sh2));
                for (uint32_t k = 0; k < rounds; ++k) {
                    const uint32_t d = 1u << k;
                    const uint32_t w = (uint32_t)__shfl((int)u, (int)(sub >= d ? lane - d : lane), 64);
                    const uint32_t y = mat_apply(mats + k * WIN_MAT_WORDS, w);
                    if (sub >= d) u ^= y;
                }
                const uint32_t cin = (uint32_t)__shfl((int)u, (int)(sub > 0 ? lane - 1 : lane), 64);
                if (sub > 0) c = cin;
            }
#pragma unroll
            for (int j = 0; j < E; ++j) {
                c = rec_reg(p, X[j] ^ (c >> p.sh2));
                if (W * j < left) buf[h + off0 + W * j] = c;
            }
            group_sync<TPS>();
            for (uint32_t p0 = 0; p0 < wc; p0 += 256) {
                uint32_t x[4], o[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t pp = p0 + 64u * i + lane;
                    const uint32_t at = h + (pp < wc ? pp : wc - 1u);
                    x[i] = buf[at];
                    o[i] = buf[at - W - 1];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = temper<F32>(tbl, x[i], o[i]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t pp = p0 + 64u * i + lane;
                    if (pp < wc) {
                        gout[done + pp] = o[i];
                        if (want_raw) raw[N + done + pp] = x[i];
                    }
                }
            }
            group_sync<TPS>();
            h += wc;
            done += wc;
        }
    }

    template <bool F32, bool LAT>
    static __device__ __forceinline__ void steps_window(const Step &p,
                                                        const uint32_t *__restrict__ prm,
                                                        uint32_t *__restrict__ buf,
                                                        gptr<uint32_t> gout, gptr<uint32_t> raw,
                                                        bool want_raw, uint64_t count,
                                                        uint32_t &h, uint64_t &done,
                                                        uint32_t lane) {
        switch (prm[P_WIN_E]) {
#define MTGP_WE(E) \
    case E:                                                                                       \
        if constexpr (LAT)                                                                        \
            steps_window_lat<F32, E>(p, prm, buf, gout, raw, want_raw, count, h, done, lane);     \
        else                                                                                      \
            steps_window_e<F32, E>(p, prm, buf, gout, raw, want_raw, count, h, done, lane);       \
        break;
            MTGP_WE(1) MTGP_WE(2) MTGP_WE(3) MTGP_WE(4)
            MTGP_WE(5) MTGP_WE(6) MTGP_WE(7) MTGP_WE(8)
#undef MTGP_WE
            default: break;
        }
    }

    // One step of KE outputs per lane (KE = ceil(S / TPS)), straight-line.
    template <bool F32, int KE>
    static __device__ __forceinline__ void body(const Step &p, uint32_t *__restrict__ buf,
                                                const uint32_t *__restrict__ tbl,
                                                gptr<uint32_t> o, gptr<uint32_t> rw,
                                                bool want_raw, uint32_t h, uint32_t S,
                                                uint32_t lane) {
        const uint32_t *q = buf + (h + lane - N);
        const uint32_t *qp = q + (p.pos - 1);
        uint32_t a[KE], b[KE], hh[KE], c[KE];
#pragma unroll
        for (int k = 0; k < KE; ++k) {
            a[k] = q[k * TPS];
            b[k] = q[k * TPS + 1];
            hh[k] = qp[k * TPS];
            c[k] = qp[k * TPS + 1];
        }
        uint32_t x[KE], r[KE];
#pragma unroll
        for (int k = 0; k < KE; ++k) {
            const uint32_t X = (a[k] & p.mask) ^ b[k];
            x[k] = rec<false>(p, tbl, xor3(X, X << p.sh1, c[k] >> p.sh2));
            r[k] = temper<F32>(tbl, x[k], hh[k]);
        }
        uint32_t *w = buf + (h + lane);
#pragma unroll
        for (int k = 0; k < KE; ++k) w[k * TPS] = x[k];
        // every k but the last is full (S > (KE-1)*TPS)
#pragma unroll
        for (int k = 0; k < KE - 1; ++k) o[k * TPS] = r[k];
        if (lane + (KE - 1) * TPS < S) o[(KE - 1) * TPS] = r[KE - 1];
        if (want_raw) {
#pragma unroll
            for (int k = 0; k < KE; ++k)
                if (lane + k * TPS < S) rw[k * TPS] = x[k];
        }
    }

    // Whole steps of S = KE rows (the same S every step), then nothing:
    // the caller finishes the partial last step.
    template <bool F32, int KE>
    static __device__ __forceinline__ void full_steps(const Step &p, uint32_t *__restrict__ buf,
                                                      const uint32_t *__restrict__ tbl,
                                                      gptr<uint32_t> gout, gptr<uint32_t> raw,
                                                      bool want_raw, uint64_t n_steps,
                                                      uint32_t S, uint32_t &h, uint64_t &done,
                                                      uint32_t lane) {
        for (uint64_t st = 0; st < n_steps; ++st) {
            maybe_compact(buf, h, SMAX, lane);
            body<F32, KE>(p, buf, tbl, gout + done + lane, raw + N + done + lane, want_raw, h,
                          S, lane);
            group_sync<TPS>();
            h += S;
            done += S;
        }
    }

    template <bool F32>
    static __device__ __forceinline__ void steps_wide(const Step &p, uint32_t *__restrict__ buf,
                                                      const uint32_t *__restrict__ tbl,
                                                      gptr<uint32_t> gout, gptr<uint32_t> raw,
                                                      bool want_raw, uint64_t count,
                                                      uint32_t &h, uint64_t &done,
                                                      uint32_t lane) {
        // full steps: W rounded down to whole 128-byte lines when wide
        uint32_t smax = p.W >= 64 ? (p.W & ~31u) : p.W;
        if (smax > (uint32_t)SMAX) smax = SMAX;
        // lanes compute every word of their rows, so keep h + SMAX inside
        // the buffer (words past S are rewritten before any read)
        const uint64_t n_full = (count - done) / smax;
        switch ((smax + TPS - 1) / TPS) {
#define MTGP_FULL(KE)                                                                       \
    case KE:                                                                                \
        if constexpr (KE <= K)                                                              \
            full_steps<F32, KE>(p, buf, tbl, gout, raw, want_raw, n_full, smax, h, done,   \
                                lane);                                                      \
        break;
            MTGP_FULL(1) MTGP_FULL(2) MTGP_FULL(3) MTGP_FULL(4)
            MTGP_FULL(5) MTGP_FULL(6) MTGP_FULL(7) MTGP_FULL(8)
#undef MTGP_FULL
            default: break;
        }
        if (done < count) {
            const uint32_t S = (uint32_t)(count - done);
            maybe_compact(buf, h, SMAX, lane);
            gptr<uint32_t> o = gout + done + lane;
            gptr<uint32_t> rw = raw + N + done + lane;
            switch ((S + TPS - 1) / TPS) {
#define MTGP_BODY(KE) \
    case KE: if constexpr (KE <= K) body<F32, KE>(p, buf, tbl, o, rw, want_raw, h, S, lane); break;
                MTGP_BODY(1) MTGP_BODY(2) MTGP_BODY(3) MTGP_BODY(4)
                MTGP_BODY(5) MTGP_BODY(6) MTGP_BODY(7) MTGP_BODY(8)
#undef MTGP_BODY
                default: break;
            }
            group_sync<TPS>();
            h += S;
            done += S;
        }
    }

    // A group of segments of one narrow stream with a linear recursion table:
    // member m on lanes [m GL, (m+1) GL), GL = 64 >> lg, each in its own part
    // of the LDS block, all in step.  A window of wn <= N-1 words per member
    // is the affine chain of steps_window_e over q = GL / W lanes per residue
    // class, E elements each; q is 1 but for W <= 4, so there is mostly no
    // scan and no second pass, and the outputs leave from the registers of
    // the chain (pieces of W words; L2 joins them to lines).  Members shorter
    // than the longest (the first segment, the last) stop storing at their
    // end, where their end state is checked or kept.  4000 mexp-3217 streams
    // of 2^18 outputs, segments alone: W = 2 2.2 TB/s (one segment per wave,
    // window scan: 0.9), W = 8 3.4 (1.2), W = 16 3.9 (1.5), W = 32 4.1 (1.9).
    template <bool F32, int E, bool SCAN>
    static __device__ __forceinline__ void steps_group(const Step &p, const GroupItem &item,
                                                       uint32_t *__restrict__ buf, uint32_t lg,
                                                       uint32_t q, uint32_t wn, uint32_t lane,
                                                       uint32_t *fail) {
        const uint32_t *tbl = buf + GBUF;
        const uint32_t *mats = tbl + 32;
        const uint32_t GL = 64u >> lg, seg = (uint32_t)GBUF >> lg;
        const uint32_t m = lane >> (6u - lg), gl = lane & (GL - 1u);
        const uint32_t W = p.W;
        const uint32_t r = SCAN ? gl / q : gl, sub = SCAN ? gl - r * q : 0u;
        const uint32_t off0 = r + W * (sub * (uint32_t)E);
        const bool ok = r < W;
        uint32_t *b = buf + m * seg;
        // this lane's member: its outputs and start state
        const uint32_t k = item.first + m;
        const uint64_t start = k == 0 ? item.prefix : (uint64_t)k * item.lseg;
        const uint64_t stop = (uint64_t)(k + 1) * item.lseg;
        const uint64_t end = stop < item.count ? stop : item.count;
        const uint32_t cnt = m < item.n ? (uint32_t)(end - start) : 0u;
        uint32_t most = cnt;
#pragma unroll
        for (int d = 8; d < 64; d <<= 1) {
            const uint32_t o = (uint32_t)__shfl_xor((int)most, d, 64);
            most = o > most ? o : most;
        }
        most = __builtin_amdgcn_readfirstlane(most);
        const uint32_t *st = reinterpret_cast<const uint32_t *>(item.states) + (uint64_t)k * N;
        if (cnt)
            for (uint32_t i = gl; i < (uint32_t)N; i += GL) b[i] = st[i];
        gptr<uint32_t> out = (gptr<uint32_t>)(reinterpret_cast<uint32_t *>(item.out)) + start;
        group_sync<TPS>();
        uint32_t h = N;
        for (uint32_t done = 0; done < most; done += wn, h += wn) {
            if (h + wn > seg) {  // the newest N words to the front, in order
                const uint32_t *src = b + (h - N);
                for (uint32_t i0 = 0; i0 < (uint32_t)N; i0 += 8 * GL) {
                    uint32_t t[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const uint32_t i = i0 + gl + GL * j;
                        t[j] = src[i < (uint32_t)N ? i : 0u];
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const uint32_t i = i0 + gl + GL * j;
                        if (i < (uint32_t)N) b[i] = t[j];
                    }
                }
                group_sync<TPS>();
                h = N;
            }
            uint32_t *w = b + h + off0;
            uint32_t X[E], v[E];
            if (ok) {
#pragma unroll
                for (int j = 0; j < E; ++j) {
                    // past the window's end only with a scan's last chunks
                    const uint32_t *s = !SCAN || off0 + W * j < wn ? w + W * j - N : b + h - N;
                    const uint32_t x0 = (s[0] & p.mask) ^ s[1];
                    X[j] = x0 ^ (x0 << p.sh1);
                }
                uint32_t c = sub == 0 ? b[h + r - W] : 0u;
                if constexpr (SCAN) {
                    uint32_t u = c;
#pragma unroll
                    for (int j = 0; j < E; ++j) u = rec<false>(p, tbl, X[j] ^ (u >> p.sh2));
#pragma unroll
                    for (int i = 0; i < GROUP_ROUNDS; ++i) {
                        const uint32_t d = 1u << i;
                        const uint32_t o = (uint32_t)__shfl((int)u, (int)(sub >= d ? lane - d : lane), 64);
                        const uint32_t y = mat_apply(mats + i * WIN_MAT_WORDS, o);
                        if (sub >= d) u ^= y;
                    }
                    const uint32_t in = (uint32_t)__shfl((int)u, (int)(sub ? lane - 1 : lane), 64);
                    if (sub) c = in;
                }
#pragma unroll
                for (int j = 0; j < E; ++j) {
                    v[j] = c = rec<false>(p, tbl, X[j] ^ (c >> p.sh2));
                    if (!SCAN || off0 + W * j < wn) w[W * j] = c;
                }
            }
            group_sync<TPS>();
            if constexpr (SCAN) {
                for (uint32_t i = gl; i < wn; i += GL)
                    if (done + i < cnt)
                        out[done + i] = temper<F32>(tbl, b[h + i], b[h + i - W - 1]);
            } else if (ok) {
                uint32_t t[E];
#pragma unroll
                for (int j = 0; j < E; ++j) t[j] = *(w + W * j - W - 1);
#pragma unroll
                for (int j = 0; j < E; ++j) t[j] = temper<F32>(tbl, v[j], t[j]);
                gptr<uint32_t> o = out + (done + off0);
                if (done + wn <= cnt) {
#pragma unroll
                    for (int j = 0; j < E; ++j) o[W * j] = t[j];
                } else {
#pragma unroll
                    for (int j = 0; j < E; ++j)
                        if (done + off0 + W * j < cnt) o[W * j] = t[j];
                }
            }
            if (cnt > done && cnt <= done + wn) {  // this member ends here
                const uint32_t *e = b + h + (cnt - done) - N;
                if (end == item.count) {
                    uint32_t *row = reinterpret_cast<uint32_t *>(item.state_out);
                    for (uint32_t i = gl; i < (uint32_t)N; i += GL) row[i] = e[i];
                } else {
                    const uint32_t *next = st + N;
                    uint32_t bad = 0;
                    for (uint32_t i = gl; i < (uint32_t)N; i += GL)
                        bad |= e[i] != next[i] ? 1u : 0u;
                    if (bad) atomicOr(fail, 1u);
                }
            }
            group_sync<TPS>();
        }
    }

    // A group of a stream with 32 < W < 64: lane l < W takes residue class l of
    // each of R members, so that R chains are in flight per lane (a single
    // segment's window of at most three elements leaves the wave waiting).
    // The same streams with W = 33 2.8 TB/s (2.0), W = 50 3.6 (2.5), W = 63
    // 3.8 (2.6).
    template <bool F32, int E, int R>
    static __device__ __forceinline__ void steps_rows(const Step &p, const GroupItem &item,
                                                      uint32_t *__restrict__ buf, uint32_t lane,
                                                      uint32_t *fail) {
        constexpr uint32_t SEG = (uint32_t)GBUF / R;
        static_assert(!GROUPS || SEG >= 2 * N, "a row holds a state and a window");
        const uint32_t *tbl = buf + GBUF;
        const uint32_t W = p.W, wn = W * E;
        const bool ok = lane < W;
        uint32_t cnt[R], most = 0;
        gptr<uint32_t> out[R];
#pragma unroll
        for (int m = 0; m < R; ++m) {
            const uint32_t k = item.first + m;
            const uint64_t start = k == 0 ? item.prefix : (uint64_t)k * item.lseg;
            const uint64_t stop = (uint64_t)(k + 1) * item.lseg;
            const uint64_t end = stop < item.count ? stop : item.count;
            cnt[m] = (uint32_t)m < item.n ? (uint32_t)(end - start) : 0u;
            most = cnt[m] > most ? cnt[m] : most;
            out[m] = (gptr<uint32_t>)(reinterpret_cast<uint32_t *>(item.out)) + start;
            const uint32_t *st = reinterpret_cast<const uint32_t *>(item.states) + (uint64_t)k * N;
            if (cnt[m])
                for (uint32_t i = lane; i < (uint32_t)N; i += 64) buf[m * SEG + i] = st[i];
        }
        group_sync<TPS>();
        uint32_t h = N;
        for (uint32_t done = 0; done < most; done += wn, h += wn) {
            if (h + wn > SEG) {  // the newest N words to the front, in order
                constexpr int C = (N + 63) / 64;
                uint32_t t[R][C];
#pragma unroll
                for (int m = 0; m < R; ++m)
#pragma unroll
                    for (int j = 0; j < C; ++j) {
                        const uint32_t i = lane + 64u * j;
                        t[m][j] = buf[m * SEG + h - N + (i < (uint32_t)N ? i : 0u)];
                    }
#pragma unroll
                for (int m = 0; m < R; ++m)
#pragma unroll
                    for (int j = 0; j < C; ++j) {
                        const uint32_t i = lane + 64u * j;
                        if (i < (uint32_t)N) buf[m * SEG + i] = t[m][j];
                    }
                group_sync<TPS>();
                h = N;
            }
            uint32_t *w = buf + h + lane;
            uint32_t X[R][E], v[R][E];
            if (ok) {
                uint32_t c[R];
#pragma unroll
                for (int m = 0; m < R; ++m) {
                    c[m] = *(w + m * SEG - W);
#pragma unroll
                    for (int j = 0; j < E; ++j) {
                        const uint32_t *s = w + m * SEG + W * j - N;
                        const uint32_t x0 = (s[0] & p.mask) ^ s[1];
                        X[m][j] = x0 ^ (x0 << p.sh1);
                    }
                }
#pragma unroll
                for (int j = 0; j < E; ++j)
#pragma unroll
                    for (int m = 0; m < R; ++m) {
                        v[m][j] = c[m] = rec<false>(p, tbl, X[m][j] ^ (c[m] >> p.sh2));
                        w[m * SEG + W * j] = c[m];
                    }
            }
            group_sync<TPS>();
            if (ok) {
                uint32_t t[R][E];
#pragma unroll
                for (int m = 0; m < R; ++m)
#pragma unroll
                    for (int j = 0; j < E; ++j) t[m][j] = *(w + m * SEG + W * j - W - 1);
#pragma unroll
                for (int m = 0; m < R; ++m)
#pragma unroll
                    for (int j = 0; j < E; ++j) t[m][j] = temper<F32>(tbl, v[m][j], t[m][j]);
#pragma unroll
                for (int m = 0; m < R; ++m) {
                    gptr<uint32_t> o = out[m] + done + lane;
                    if (done + wn <= cnt[m]) {
#pragma unroll
                        for (int j = 0; j < E; ++j) o[W * j] = t[m][j];
                    } else {
#pragma unroll
                        for (int j = 0; j < E; ++j)
                            if (done + lane + W * j < cnt[m]) o[W * j] = t[m][j];
                    }
                }
            }
#pragma unroll
            for (int m = 0; m < R; ++m)
                if (cnt[m] > done && cnt[m] <= done + wn) {  // this member ends here
                    const uint32_t k = item.first + m;
                    const uint32_t *e = buf + m * SEG + h + (cnt[m] - done) - N;
                    if ((uint64_t)(k + 1) * item.lseg >= item.count) {
                        uint32_t *row = reinterpret_cast<uint32_t *>(item.state_out);
                        for (uint32_t i = lane; i < (uint32_t)N; i += 64) row[i] = e[i];
                    } else {
                        const uint32_t *next = reinterpret_cast<const uint32_t *>(item.states) +
                                               (uint64_t)(k + 1) * N;
                        uint32_t bad = 0;
                        for (uint32_t i = lane; i < (uint32_t)N; i += 64)
                            bad |= e[i] != next[i] ? 1u : 0u;
                        if (bad) atomicOr(fail, 1u);
                    }
                }
            group_sync<TPS>();
        }
    }

    template <bool F32>
    static __device__ __forceinline__ void run_group(const uint32_t *__restrict__ prm,
                                                     const GroupItem &item,
                                                     uint32_t *__restrict__ buf, uint32_t lane) {
        Step p = load_step(prm);
        const uint32_t lg = (uint32_t)group_log(p.W), GL = 64u >> lg, q = GL / p.W;
        uint32_t *tbl = buf + GBUF;
        group_sync<TPS>();  // the previous user of this buffer is done with it
        if (lane < 16) {
            tbl[lane] = prm[P_REC + lane];
            tbl[16 + lane] = prm[(F32 ? P_FLT : P_TMP) + lane];
        }
        uint32_t *fail = &reinterpret_cast<ReqRec *>(item.rec)->failed;
        if (p.W > 32u) {
            group_sync<TPS>();
#define MTGP_GR(E)                                                        \
    case E:                                                               \
        if (item.n > 1u) steps_rows<F32, E, GROUP_ROWS>(p, item, buf, lane, fail); \
        else steps_rows<F32, E, 1>(p, item, buf, lane, fail);             \
        break;
            switch ((N - 1) / p.W) {  // E W < N, W > 32, N <= 128
                MTGP_GR(1) MTGP_GR(2) MTGP_GR(3)
                default: break;
            }
#undef MTGP_GR
            return;
        }
        if (q > 1u) {
            for (uint32_t i = lane; i < (uint32_t)(GROUP_ROUNDS * WIN_MAT_WORDS); i += 64)
                tbl[32 + i] = prm[P_GRP_MAT + i];
            // W q E words, E = 8 (W <= 4, q = 8 / W)
            steps_group<F32, GROUP_E, true>(p, item, buf, lg, q, p.W * q * GROUP_E, lane, fail);
            return;
        }
        switch ((N - 1) / p.W) {  // whole windows of E W words, W <= 32 and N > 96
#define MTGP_GE(E) \
    case E: steps_group<F32, E, false>(p, item, buf, lg, 1u, p.W * E, lane, fail); break;
            MTGP_GE(3) MTGP_GE(4) MTGP_GE(5) MTGP_GE(6) MTGP_GE(7)
#undef MTGP_GE
            default: steps_group<F32, 8, false>(p, item, buf, lg, 1u, p.W * 8, lane, fail); break;
        }
    }

    static __device__ __forceinline__ Step load_step(const uint32_t *__restrict__ prm) {
        Step p;
        p.pos = prm[P_POS];
        p.sh1 = prm[P_SH1];
        p.sh2 = prm[P_SH2];
        p.mask = prm[P_MASK];
        p.W = N - p.pos;
        p.rb0 = prm[P_RB + 0];
        p.rb1 = prm[P_RB + 1];
        p.rb2 = prm[P_RB + 2];
        p.rb3 = prm[P_RB + 3];
        return p;
    }

    // Advance one stream by item.count outputs.  A MODE_VERIFY item that
    // ends in a state other than item.verify sets *fail.  RAW: the
    // MODE_RAW word dump is compiled in (prefix kernels only); LAT: narrow
    // streams take the window for a wave that runs nearly alone.
    template <bool F32, bool RAW, bool LAT>
    static __device__ __forceinline__ void run(const uint32_t *__restrict__ prm,
                                               const BatchItem &item,
                                               uint32_t *__restrict__ buf, uint32_t lane,
                                               uint32_t *fail, uint32_t win_below) {
        // a stream takes the window path when the host gave it window data
        const bool win = TPS == 64 && prm[P_WIN_E] != 0u && prm[P_W] < win_below;
        uint32_t *__restrict__ tbl = buf + (win ? WBUF : BUF);
        const Step p = load_step(prm);
        const uint32_t lin = prm[P_LIN];
        const uint64_t count = item.count;
        const uint32_t *st_in = reinterpret_cast<const uint32_t *>(item.state_in);
        uint32_t *st_out = reinterpret_cast<uint32_t *>(item.state_out);
        gptr<uint32_t> raw = (gptr<uint32_t>)(reinterpret_cast<uint32_t *>(item.raw));
        gptr<uint32_t> gout = (gptr<uint32_t>)(reinterpret_cast<uint32_t *>(item.out));
        const bool want_raw = RAW && (item.mode & MODE_RAW) != 0;

        group_sync<TPS>();  // previous user of this buffer is done with it
        for (uint32_t i = lane; i < N; i += TPS) {
            const uint32_t v = st_in[i];
            buf[i] = v;
            if (want_raw) raw[i] = v;
        }
        if (lane < 16) {
            tbl[lane] = prm[P_REC + lane];
            tbl[16 + lane] = prm[(F32 ? P_FLT : P_TMP) + lane];
        }
        group_sync<TPS>();

        uint32_t h = N;  // buffer index of the next new word
        uint64_t done = 0;
        if (win) {
            steps_window<F32, LAT>(p, prm, buf, gout, raw, want_raw, count, h, done, lane);
        } else if (TPS == 64 && p.W < 64) {
            if (lin)
                steps_small<F32, true>(p, buf, tbl, gout, raw, want_raw, count, h, done, lane);
            else
                steps_small<F32, false>(p, buf, tbl, gout, raw, want_raw, count, h, done, lane);
        } else {
            steps_wide<F32>(p, buf, tbl, gout, raw, want_raw, count, h, done, lane);
        }
        group_sync<TPS>();
        if (st_out != nullptr)
            for (uint32_t i = lane; i < N; i += TPS) st_out[i] = buf[h - N + i];
        if ((item.mode & MODE_VERIFY) && fail != nullptr) {
            // the end state must equal the next segment's jumped start state
            const uint32_t *ref = reinterpret_cast<const uint32_t *>(item.verify);
            uint32_t bad = 0;
            for (uint32_t i = lane; i < N; i += TPS) bad |= (buf[h - N + i] != ref[i]) ? 1u : 0u;
            if (bad) atomicOr(fail, 1u);
        }
    }
};

// Plain mode (items == nullptr): item i is stream i, advanced in place in
// its state row by plain_count outputs written at plain_out + i*plain_count.
struct PlainArgs {
    uint32_t *states;
    uint32_t stride;
    uint32_t mode;
    uint32_t *out;
    uint64_t count;
};

__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Value of lane 0 (wave) or thread 0 (workgroup) for the whole group.
template <int TPS>
__device__ __forceinline__ uint32_t group_first(uint32_t v, uint32_t *slot) {
    if constexpr (TPS == 64) {
        return __builtin_amdgcn_readfirstlane(v);
    } else {
        __syncthreads();
        if (threadIdx.x == 0) *slot = v;
        __syncthreads();
        return *slot;
    }
}

// The work loop shared by the generation kernels: claim an item (or take
// stream `it` in plain mode), run it, raise its completion flag.
template <int N, int TPS, int K, int WPB, bool RAW, bool LAT, bool GRP>
__device__ __forceinline__ void gen_body(const uint32_t *__restrict__ params,
                                         const BatchItem *__restrict__ items, uint32_t n_items,
                                         uint32_t *__restrict__ counter, uint32_t persistent,
                                         uint32_t win_below, PlainArgs plain) {
    using C = Core<N, TPS, K, GRP>;
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t s_claim;
    const uint32_t wave =
        (TPS == 64) ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0u;
    const uint32_t lane = (TPS == 64) ? (threadIdx.x & 63u) : threadIdx.x;
    uint32_t *buf = lds + wave * C::LDS_WORDS;
    const uint32_t n_groups = gridDim.x * (TPS == 64 ? WPB : 1);
    uint32_t it = blockIdx.x * (TPS == 64 ? WPB : 1) + wave;

    while (true) {
        if (persistent) {
            uint32_t v = 0;
            if (lane == 0) v = atomicAdd(counter, 1u);
            it = group_first<TPS>(v, &s_claim);
        }
        if (it >= n_items) break;
        BatchItem item;
        if (items != nullptr) {
            item = items[it];
        } else {
            uint32_t *row = plain.states + (uint64_t)it * plain.stride;
            item.stream = it;
            item.mode = plain.mode;
            item.count = plain.count;
            item.out = (uint64_t)(uintptr_t)(plain.out + (uint64_t)it * plain.count);
            item.state_in = item.state_out = (uint64_t)(uintptr_t)row;
            item.raw = item.verify = item.rec = item.flag = 0;
        }
        if (GRP && (item.mode & MODE_GROUP)) {
            if constexpr (GRP) {
                const GroupItem g = *reinterpret_cast<const GroupItem *>(items + it);
                const uint32_t *prm = params + (uint64_t)g.stream * P_WORDS;
                if (g.mode & MODE_F32) C::template run_group<true>(prm, g, buf, lane);
                else C::template run_group<false>(prm, g, buf, lane);
            }
        } else if (item.count > 0) {
            const uint32_t *prm = params + (uint64_t)item.stream * P_WORDS;
            uint32_t *fail = (item.mode & MODE_VERIFY)
                                 ? &reinterpret_cast<ReqRec *>(item.rec)->failed
                                 : nullptr;
            if (item.mode & MODE_F32)
                C::template run<true, RAW, LAT>(prm, item, buf, lane, fail, win_below);
            else
                C::template run<false, RAW, LAT>(prm, item, buf, lane, fail, win_below);
        }
        if (item.flag != 0) {
            // Publish completion of the request to the host: every lane's
            // output and state stores are made visible system-wide first.
            // (a wave's lanes all store the flag: with a store by lane 0 alone
            // the compiler may split the claim loop by lane.)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
            group_sync<TPS>();
            if (TPS == 64 || lane == 0)
                __hip_atomic_store(reinterpret_cast<uint32_t *>(item.flag), 1u, __ATOMIC_RELEASE,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
        }
        if (!persistent) it += n_groups;
    }
}

// Segments of a batch, whole unsplit requests and plain calls; GRP: groups
// among them.
template <int N, int TPS, int K, int WPB, bool GRP>
__global__ void __launch_bounds__(TPS == 64 ? 64 * WPB : TPS)
gen_kernel(const uint32_t *__restrict__ params, const BatchItem *__restrict__ items,
           uint32_t n_items, uint32_t *__restrict__ counter, uint32_t persistent,
           uint32_t win_below, PlainArgs plain) {
    gen_body<N, TPS, K, WPB, false, false, GRP>(params, items, n_items, counter, persistent,
                                                win_below, plain);
}

// Plain calls of few streams: one wave per stream with room for longer runs
// between compactions, and the latency-bound window.
template <int N>
__global__ void __launch_bounds__(256)
few_kernel(const uint32_t *__restrict__ params, const BatchItem *__restrict__ items,
           uint32_t n_items, uint32_t *__restrict__ counter, uint32_t persistent,
           uint32_t win_below, PlainArgs plain) {
    gen_body<N, 64, 8, 4, false, true, false>(params, items, n_items, counter, persistent,
                                              win_below, plain);
}

// Segments and whole requests of a batch with fewer items than the chip has
// SIMDs: a wave that runs alone spends a step issuing the instructions of
// its rows (four rows of 64 outputs 980 cycles, of which some 300 are the
// chain), so streams of wide steps are run by whole workgroups, a row or a
// few per wave.  The workgroups first claim the wide items, then their waves
// the others.  No completion flags: requests that carry one are the server's,
// whose batches are never sparse.
constexpr int wide_k(int N) { return N <= 400 ? 1 : N <= 800 ? 2 : 4; }

template <int N>
constexpr int sparse_lds_words() {
    const int a = 4 * Core<N, 64, 8>::LDS_WORDS, b = Core<N, 256, wide_k(N)>::LDS_WORDS;
    return (a > b ? a : b) + 4;
}

template <int N>
__global__ void __launch_bounds__(256)
sparse_kernel(const uint32_t *__restrict__ params, const BatchItem *__restrict__ items,
              uint32_t n_wide, uint32_t n_items, uint32_t *__restrict__ wide_counter,
              uint32_t *__restrict__ counter, uint32_t win_below) {
    using B = Core<N, 256, wide_k(N)>;
    using A = Core<N, 64, 8>;
    extern __shared__ uint32_t lds[];
    uint32_t &s_claim = lds[sparse_lds_words<N>() - 4];
    while (true) {  // wide items, one per workgroup
        __syncthreads();
        if (threadIdx.x == 0) s_claim = atomicAdd(wide_counter, 1u);
        __syncthreads();
        const uint32_t it = __builtin_amdgcn_readfirstlane(s_claim);
        if (it >= n_wide) break;
        const BatchItem item = items[it];
        const uint32_t *prm = params + (uint64_t)item.stream * P_WORDS;
        uint32_t *fail = (item.mode & MODE_VERIFY) ? &reinterpret_cast<ReqRec *>(item.rec)->failed
                                                   : nullptr;
        if (item.mode & MODE_F32)
            B::template run<true, false, false>(prm, item, lds, threadIdx.x, fail, 0u);
        else
            B::template run<false, false, false>(prm, item, lds, threadIdx.x, fail, 0u);
    }
    __syncthreads();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t *buf = lds + wave * A::LDS_WORDS;
    while (true) {  // the others, one per wave
        uint32_t v = 0;
        if (lane == 0) v = atomicAdd(counter, 1u);
        const uint32_t it = n_wide + __builtin_amdgcn_readfirstlane(v);
        if (it >= n_items) break;
        const BatchItem item = items[it];
        const uint32_t *prm = params + (uint64_t)item.stream * P_WORDS;
        uint32_t *fail = (item.mode & MODE_VERIFY) ? &reinterpret_cast<ReqRec *>(item.rec)->failed
                                                   : nullptr;
        if (item.mode & MODE_F32)
            A::template run<true, false, true>(prm, item, buf, lane, fail, win_below);
        else
            A::template run<false, false, true>(prm, item, buf, lane, fail, win_below);
    }
}

// Outputs per lane and step of the prefix kernel (the default tuning's).
__host__ __device__ constexpr int prefix_k(int N) { return N <= 400 ? 4 : 8; }

// The word runs jump-ahead planning takes its polynomials from: one wave
// per item, four waves per workgroup.
template <int N>
__global__ void __launch_bounds__(256)
prefix_kernel(const uint32_t *__restrict__ params, const BatchItem *__restrict__ items,
              uint32_t n_items, uint32_t *__restrict__ counter, uint32_t persistent,
              uint32_t win_below, PlainArgs plain) {
    gen_body<N, 64, prefix_k(N), 4, true, true, false>(params, items, n_items, counter,
                                                       persistent, win_below, plain);
}

// Request checks of split requests (MODE_FIXUP items), after every segment
// has finished.  If a segment started from a wrong jumped state (the
// stream's state lay outside the orbit its polynomial annihilates), the
// whole request is regenerated in order from its start state and logged.
// That is rare, so a wave looks at `per_wave` requests at once, one per
// lane (10,000 requests: 5 us against 107 us with a claim per request).
// Record fields are loaded from writable memory, so they are made
// wave-uniform explicitly.
template <int N>
__global__ void __launch_bounds__(256)
check_kernel(const uint32_t *__restrict__ params, const BatchItem *__restrict__ items,
             uint32_t n_items, uint32_t per_wave, uint32_t *__restrict__ err,
             uint32_t win_below) {
    using C = Core<N, 64, 1>;
    extern __shared__ uint32_t lds[];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t i = (blockIdx.x * 4 + wave) * per_wave + lane;
    uint64_t rec_addr = 0, flag = 0;
    uint32_t failed = 0;
    if (lane < per_wave && i < n_items) {
        rec_addr = items[i].rec;
        flag = items[i].flag;
        failed = __hip_atomic_load(&reinterpret_cast<const ReqRec *>(rec_addr)->failed,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    uint64_t todo = __builtin_amdgcn_ballot_w64(failed != 0u);
    while (todo) {
        const int l = __builtin_ctzll(todo);
        todo &= todo - 1;
        const uint64_t addr = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(
                                   (int)(uint32_t)(rec_addr >> 32), l) << 32) |
                              (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)rec_addr, l);
        const ReqRec *rec = reinterpret_cast<const ReqRec *>(addr);
        BatchItem item;
        item.stream = __builtin_amdgcn_readfirstlane(rec->stream);
        item.mode = __builtin_amdgcn_readfirstlane(rec->mode);
        item.count = uniform64(rec->count);
        item.out = uniform64(rec->out);
        item.state_in = uniform64(rec->orig);
        item.state_out = uniform64(rec->row);
        item.raw = item.verify = 0;
        if (lane == 0) {
            atomicAdd(err, 1u);
            const uint32_t slot = atomicAdd(err + 1, 1u);
            if (slot < (uint32_t)HDR_LOG_MAX) err[2 + slot] = item.stream;
        }
        const uint32_t *prm = params + (uint64_t)item.stream * P_WORDS;
        uint32_t *buf = lds + wave * C::LDS_WORDS;
        if (item.mode & MODE_F32)
            C::template run<true, false, false>(prm, item, buf, lane, nullptr, win_below);
        else
            C::template run<false, false, false>(prm, item, buf, lane, nullptr, win_below);
    }
    if (__builtin_amdgcn_ballot_w64(flag != 0)) {
        // publish completion to the host, after every lane's stores
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
        group_sync<64>();
        if (flag != 0)
            __hip_atomic_store(reinterpret_cast<uint32_t *>(flag), 1u, __ATOMIC_RELEASE,
                               __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Jump evaluation: out_j[m] = XOR over the set bits i < D of g_j of r[i+m]
// with r[n] = raw[1+n], for m < M: the product of a binary Hankel matrix of
// words with the coefficient vectors of the block's jumps.
//
// Outputs are cut into T tiles of 128 words and coefficients into chunks of
// T parts of 128, so that a chunk is a T x T block matrix whose block (a, b)
// is the Hankel block R_{a+b} of words r[128 (a+b) ..].  With
//   M_ab = R_{a+b} (g_a + g_b)   and   D_a = (sum over b of R_{a+b}) g_a
// every output tile is y_a = D_a + the sum over b != a of M_ab, and M_ab
// serves y_a and y_b: T (T+1) / 2 block products instead of T^2.
//
// A block product takes its coefficients four at a time: for a nibble value
// v of the coefficients 4c..4c+3 a jump adds Q_v[4c+m], where Q_v[n] is the
// XOR over the set bits j of v of w[n+j], w the 256 words of the block (for
// D_a the XOR of T such runs).  The workgroup builds the planes Q_1..Q_15
// in LDS (plane 0 stays zero, so lookups are branch-free) while its waves
// look up the previous product's; a half-wave covers a tile's 128 words of
// one jump, four words per lane and 16-byte read, two nibbles per
// three-input XOR.  Where the block holds few jumps, two or four half-waves
// share a jump's nibbles and are summed at the end.
//
// Bound by the 16-byte LDS reads and the vector work around them (four
// operations per read): the prefix-and-jump launch of 128 x 2^24 mexp-11213
// outputs takes 464-520 us (646-750 with T^2 block products over 512-word
// tiles), of 4096 x 2^20 mexp-23209 490 us (650).
constexpr int JUMP_WAVES = 4;
constexpr int JUMP_PLANE = 2 * JUMP_TILE;                 // plane length (words)
constexpr int JUMP_PLANES_WORDS = 16 * JUMP_PLANE;        // one product's planes
static_assert(JUMP_BLOCK == 2 * JUMP_WAVES, "one jump per half-wave");
__host__ __device__ constexpr int jump_lds_words(int T) {
    // two sets of planes, two chunks of 2T tiles of words
    return 2 * JUMP_PLANES_WORDS + 2 * 2 * T * JUMP_TILE;
}

typedef uint32_t jv4 __attribute__((ext_vector_type(4)));

// 16 bytes of the plane that bits s .. s+3 of `bits` name, at LDS address
// col + off in plane 0.
__device__ __forceinline__ jv4 plane_read(uint32_t col, uint32_t bits, int s, int off) {
    const uint32_t v = s >= 10 ? bits >> (s - 10) : bits << (10 - s);
    return *reinterpret_cast<lptr<const jv4>>((uintptr_t)(((v & 0x3C00u) | col) + off));
}

// WPP: coefficient words (of the four of a part) one half-wave takes.
template <int T, int WPP>
__device__ __forceinline__ void jump_block(const JumpBlock &jb, uint32_t *__restrict__ lds,
                                           uint32_t wave, uint32_t lane) {
    constexpr uint32_t PARTS = 4 / WPP;
    constexpr uint32_t CHUNK = T * JUMP_TILE;             // coefficients per chunk
    constexpr uint32_t STAGE = 2 * T * JUMP_TILE;         // words a chunk reads
    uint32_t *planes = lds;
    uint32_t *stage = lds + 2 * JUMP_PLANES_WORDS;
    const uint32_t tid = wave * 64 + lane, l32 = lane & 31u;
    const uint32_t worker = 2 * wave + (lane >> 5);
    const uint32_t jump = worker / PARTS, part = worker % PARTS;
    const bool wave_active = (2 * wave) / PARTS < jb.n_jumps;  // uniform
    gptr<const uint32_t> r = (gptr<const uint32_t>)(reinterpret_cast<const uint32_t *>(jb.raw)) + 1;
    gptr<const uint32_t> g = (gptr<const uint32_t>)(reinterpret_cast<const uint32_t *>(jb.poly)) +
                             (uint64_t)(jump < jb.n_jumps ? jump : 0u) * jb.poly_stride +
                             part * WPP;
    const uint32_t pw = jb.poly_stride, rlen = jb.nbits + jb.m;
    const uint32_t n_chunks = (jb.nbits + CHUNK - 1) / CHUNK;

    uint32_t raw[T];                                      // this thread's words of a chunk to come
    auto load_raw = [&](uint32_t c) {
        gptr<const uint32_t> p = r + c * CHUNK + tid;
        if (c * CHUNK + STAGE <= rlen) {
#pragma unroll
            for (int k = 0; k < T; ++k) raw[k] = p[256 * k];
        } else {
#pragma unroll
            for (int k = 0; k < T; ++k) {
                raw[k] = 0u;
                if (c * CHUNK + tid + 256u * k < rlen) raw[k] = p[256 * k];
            }
        }
    };
    auto store_raw = [&](uint32_t c) {
#pragma unroll
        for (int k = 0; k < T; ++k) stage[(c & 1u) * STAGE + tid + 256u * k] = raw[k];
    };
    uint32_t cw[T][WPP], cn[T][WPP];                      // coefficients: this chunk's, the next's
    auto load_coeffs = [&](uint32_t c) {
        gptr<const uint32_t> p = g + c * (CHUNK / 32);
        if ((c + 1) * (CHUNK / 32) <= pw) {
#pragma unroll
            for (int a = 0; a < T; ++a)
#pragma unroll
                for (int e = 0; e < WPP; ++e) cn[a][e] = p[4 * a + e];
        } else {
#pragma unroll
            for (int a = 0; a < T; ++a)
#pragma unroll
                for (int e = 0; e < WPP; ++e) {
                    cn[a][e] = 0u;
                    if (c * (CHUNK / 32) + 4u * a + part * WPP + e < pw) cn[a][e] = p[4 * a + e];
                }
        }
    };
    const uint32_t m1 = wave & 1u ? ~0u : 0u, m2 = wave & 2u ? ~0u : 0u;
    // planes 4 wave .. 4 wave + 3 of product (a, b) of chunk c; lane i makes
    // the words 4i .. 4i+3 of each (the last four are never read)
    auto build = [&](uint32_t c, int a, int b, uint32_t *pl) {
        if (lane == 63u) return;
        const jv4 *src = reinterpret_cast<const jv4 *>(stage + (c & 1u) * STAGE) + lane;
        constexpr int TV = JUMP_TILE / 4;
        jv4 lo, hi;
        if (a != b) {
            lo = src[(a + b) * TV];
            hi = src[(a + b) * TV + 1];
        } else {
            lo = src[a * TV];
            hi = src[a * TV + 1];
#pragma unroll
            for (int k = 1; k < T; ++k) {
                lo ^= src[(a + k) * TV];
                hi ^= src[(a + k) * TV + 1];
            }
        }
        const jv4 w1 = {lo[1], lo[2], lo[3], hi[0]}, w2 = {lo[2], lo[3], hi[0], hi[1]},
                  w3 = {lo[3], hi[0], hi[1], hi[2]};
        const jv4 h = (w2 & m1) ^ (w3 & m2);
        jv4 *dst = reinterpret_cast<jv4 *>(pl + 4 * wave * JUMP_PLANE) + lane;
        dst[0] = h;
        dst[JUMP_PLANE / 4] = h ^ lo;
        dst[2 * (JUMP_PLANE / 4)] = h ^ w1;
        dst[3 * (JUMP_PLANE / 4)] = h ^ lo ^ w1;
    };

    jv4 acc[T];
#pragma unroll
    for (int a = 0; a < T; ++a) acc[a] = jv4{0u, 0u, 0u, 0u};
    load_raw(0);
    load_coeffs(0);
    __syncthreads();                                      // the previous block's LDS is free
    store_raw(0);
    if (n_chunks > 1) load_raw(1);
    __syncthreads();
    build(0, 0, 0, planes);
    uint32_t flip = 0;                                    // planes of the product looked up next
    for (uint32_t c = 0; c < n_chunks; ++c) {
#pragma unroll
        for (int a = 0; a < T; ++a)
#pragma unroll
            for (int e = 0; e < WPP; ++e) cw[a][e] = cn[a][e];
        const bool more = c + 1 < n_chunks;
        if (more) {
            // stage[(c+1) & 1] was last read before the previous barrier
            store_raw(c + 1);
            load_coeffs(c + 1);
            if (c + 2 < n_chunks) load_raw(c + 2);
        }
#pragma unroll
        for (int a = 0; a < T; ++a) {
#pragma unroll
            for (int b = a; b < T; ++b) {
                uint32_t *now = planes + flip;
                flip ^= (uint32_t)JUMP_PLANES_WORDS;
                __syncthreads();  // `now` is built, the other set no longer read
                if (b + 1 < T) build(c, a, b + 1, planes + flip);
                else if (a + 1 < T) build(c, a + 1, a + 1, planes + flip);
                else if (more) build(c + 1, 0, 0, planes + flip);
                if (wave_active) {
                    // LDS byte address of the half-wave's first lookup in plane 0;
                    // plane v lies v << 10 bytes on, bits that are zero here (the
                    // planes start at LDS address 0 and 16 KB)
                    const uint32_t col = (uint32_t)(uintptr_t)(lptr<uint32_t>)now + 16u * l32 +
                                         part * (WPP * 128);
                    jv4 y = jv4{0u, 0u, 0u, 0u};
#pragma unroll
                    for (int e = 0; e < WPP; ++e) {
                        const uint32_t bits = a == b ? cw[a][e] : cw[a][e] ^ cw[b][e];
                        jv4 q[8];  // eight reads in flight
#pragma unroll
                        for (int k = 0; k < 8; ++k)
                            q[k] = plane_read(col, bits, 4 * k, 128 * e + 16 * k);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int k = 0; k < 8; k += 2)
#pragma unroll
                            for (int i = 0; i < 4; ++i) y[i] = xor3(y[i], q[k][i], q[k + 1][i]);
                    }
                    acc[a] ^= y;
                    if (a != b) acc[b] ^= y;
                }
            }
        }
    }
    uint32_t *out = reinterpret_cast<uint32_t *>(jb.out);
    if constexpr (PARTS == 1) {
        if (jump < jb.n_jumps) {
            gptr<uint32_t> o = (gptr<uint32_t>)(out + (uint64_t)jump * jb.out_stride);
#pragma unroll
            for (int a = 0; a < T; ++a)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t m = JUMP_TILE * a + 4 * l32 + i;
                    if (m < jb.m) o[m] = acc[a][i];
                }
        }
    } else {
        __syncthreads();                                  // the planes are no longer read
        jv4 *sum = reinterpret_cast<jv4 *>(planes);
#pragma unroll
        for (int a = 0; a < T; ++a) sum[(worker * T + a) * (JUMP_TILE / 4) + l32] = acc[a];
        __syncthreads();
        const uint32_t *w = planes;
        for (uint32_t j = 0; j < jb.n_jumps; ++j) {
            gptr<uint32_t> o = (gptr<uint32_t>)(out + (uint64_t)j * jb.out_stride);
            for (uint32_t m = tid; m < jb.m; m += 64 * JUMP_WAVES) {
                uint32_t v = 0;
#pragma unroll
                for (uint32_t k = 0; k < PARTS; ++k) v ^= w[(j * PARTS + k) * CHUNK + m];
                o[m] = v;
            }
        }
    }
}

// Half-waves per jump by the jumps of the block, whose fields are made
// wave-uniform explicitly (they are loaded from writable memory).
template <int T>
__device__ __forceinline__ void jump_any(const JumpBlock &b, uint32_t *__restrict__ lds,
                                         uint32_t wave, uint32_t lane) {
    JumpBlock jb;
    jb.raw = uniform64(b.raw);
    jb.poly = uniform64(b.poly);
    jb.out = uniform64(b.out);
    jb.poly_stride = __builtin_amdgcn_readfirstlane(b.poly_stride);
    jb.out_stride = __builtin_amdgcn_readfirstlane(b.out_stride);
    jb.nbits = __builtin_amdgcn_readfirstlane(b.nbits);
    jb.m = __builtin_amdgcn_readfirstlane(b.m);
    jb.n_jumps = __builtin_amdgcn_readfirstlane(b.n_jumps);
    if (jb.n_jumps <= 2u) jump_block<T, 1>(jb, lds, wave, lane);
    else if (jb.n_jumps <= 4u) jump_block<T, 2>(jb, lds, wave, lane);
    else jump_block<T, 4>(jb, lds, wave, lane);
}

// Jump evaluation alone (the planning checks of jump-ahead polynomials).
template <int T>
__global__ void __launch_bounds__(64 * JUMP_WAVES)
jump_kernel(const JumpBlock *__restrict__ blocks, uint32_t n_blocks) {
    extern __shared__ uint32_t lds[];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t blk = blockIdx.x; blk < n_blocks; blk += gridDim.x)
        jump_any<T>(blocks[blk], lds, wave, lane);
}

// Waits (a whole wave, every lane reading the same flag) until *flag is
// nonzero; gives up after a bound far above any legitimate wait, counting
// the give-up in *timeouts (the repair count: a jump evaluated too early
// fails its segment check, and the request is regenerated).  The flag value
// is made wave-uniform so that the loop exit is uniform.
__device__ __forceinline__ void wait_flag(const uint32_t *flag, uint32_t *timeouts,
                                          uint32_t lane) {
    for (uint32_t spins = 0;; ++spins) {
        const uint32_t f = __builtin_amdgcn_readfirstlane(
            __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (f != 0u) break;
        if (spins > (1u << 24)) {  // seconds of s_sleep
            atomicAdd(timeouts, lane == 0 ? 1u : 0u);
            break;
        }
        __builtin_amdgcn_s_sleep(8);
    }
}

// Prefix items and jump blocks of a batch in one persistent launch.  Every
// wave first claims prefix items (one wave each, RAW: they dump the words
// the jumps read); once the prefix counter is exhausted (every prefix has
// been claimed by a running wave) the workgroup claims jump blocks, each of
// which waits for its stream's prefix flag.  A jump block waits only on a
// prefix claimed before any block, so every wait ends.
struct PJArgs {
    const uint32_t *params;
    const BatchItem *prefix;  // nP prefix items
    uint32_t nP;
    const JumpBlock *jumps;   // nJ jump blocks
    uint32_t nJ;
    uint32_t *pflag;          // per prefix item: set to 1 when its words are stored
    uint32_t *hdr;            // workspace header (claim counters, timeouts)
    uint32_t win_below;
};

// LDS words: the prefix buffers of the waves, or a jump block's; then the
// claim word.  No static LDS: the planes are read with 16-byte LDS loads,
// and a static word would move the dynamic region to offset 4.
template <int N>
__host__ __device__ constexpr int pj_lds_words() {
    const int pre = JUMP_WAVES * Core<N, 64, 4>::LDS_WORDS, jmp = jump_lds_words(jump_tiles(N));
    return (pre > jmp ? pre : jmp) + 4;
}

template <int N>
__global__ void __launch_bounds__(64 * JUMP_WAVES) pj_kernel(PJArgs a) {
    using C = Core<N, 64, 4>;
    extern __shared__ uint32_t lds[];
    uint32_t &s_claim = lds[pj_lds_words<N>() - 4];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t *buf = lds + wave * C::LDS_WORDS;
    while (true) {  // prefix items, one per wave
        uint32_t v = 0;
        if (lane == 0) v = atomicAdd(a.hdr + 0, 1u);
        const uint32_t it = __builtin_amdgcn_readfirstlane(v);
        if (it >= a.nP) break;
        const BatchItem item = a.prefix[it];
        const uint32_t *prm = a.params + (uint64_t)item.stream * P_WORDS;
        if (item.mode & MODE_F32)
            C::template run<true, true, true>(prm, item, buf, lane, nullptr, a.win_below);
        else
            C::template run<false, true, true>(prm, item, buf, lane, nullptr, a.win_below);
        // every lane stores the flag: a lane-0-only store here lets the
        // compiler split the claim loop by lane
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __hip_atomic_store(a.pflag + it, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    while (true) {  // jump blocks, one per workgroup
        __syncthreads();  // (first: every wave is done with its prefix buffer)
        if (threadIdx.x == 0) s_claim = atomicAdd(a.hdr + HDR_J_CLAIM, 1u);
        __syncthreads();
        const uint32_t blk = __builtin_amdgcn_readfirstlane(s_claim);
        if (blk >= a.nJ) break;
        const JumpBlock jb = a.jumps[blk];
        const uint32_t dep = __builtin_amdgcn_readfirstlane(jb.dep);
        if (wave == 0) wait_flag(a.pflag + dep, a.hdr + HDR_ERR, lane);
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        jump_any<jump_tiles(N)>(jb, lds, wave, lane);
    }
}

template <int N>
static hipError_t launch_pj_n(const PJArgs &a, int num_cus, hipStream_t s) {
    constexpr int lds = pj_lds_words<N>() * 4;
    static bool attr_set = false;  // benign race: idempotent attribute
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)pj_kernel<N>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const uint32_t work = a.nP + a.nJ;
    int grid = (int)(work > 0 ? work : 1);
    const int cap = num_cus * (160 * 1024 / lds);  // workgroups that fit the CUs' LDS
    if (grid > cap) grid = cap;
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(pj_kernel<N>, dim3(grid), dim3(64 * JUMP_WAVES), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_prefix_jumps(int n_words, const BatchItem *prefix, uint32_t nP,
                               const JumpBlock *jumps, uint32_t nJ, uint32_t *pflag,
                               const uint32_t *params, uint32_t *hdr, uint32_t win_below,
                               int num_cus, hipStream_t s) {
    PJArgs a{params, prefix, nP, jumps, nJ, pflag, hdr, win_below};
    switch (n_words) {
        case 101: return launch_pj_n<101>(a, num_cus, s);
        case 351: return launch_pj_n<351>(a, num_cus, s);
        case 726: return launch_pj_n<726>(a, num_cus, s);
        case 1391: return launch_pj_n<1391>(a, num_cus, s);
        default: return hipErrorInvalidValue;
    }
}

size_t prefix_jump_lds_bytes(int n_words) {
    switch (n_words) {
        case 101: return 4 * pj_lds_words<101>();
        case 351: return 4 * pj_lds_words<351>();
        case 726: return 4 * pj_lds_words<726>();
        case 1391: return 4 * pj_lds_words<1391>();
        default: return 0;
    }
}

// Seeding: one lane per stream runs the N-step initialisation recurrence, a
// serial chain of a shift, an XOR and a 32-bit multiply-add per word.  The
// chain bounds the kernel, so the stores must not: a wave seeds SEED_STREAMS
// streams on its first lanes into an LDS tile of SEED_TILE words each and
// then stores the tile a row at a time, SEED_TILE consecutive words of one
// stream per instruction (a lane storing its own word touches one cache
// line per lane and word).  Few streams per wave, so that a thousand of
// them reach 64 CUs.  1024 mexp-44497 streams 28 us (20 ns per word of the
// chain; a lane storing its own words: 182 us), 1000 mexp-3217 streams 4.9
// (14.5), 128 mexp-11213 streams 8.6-10.6 (24-29).
constexpr uint32_t SEED_STREAMS = 16;
constexpr uint32_t SEED_TILE = 64;

__global__ void __launch_bounds__(64)
seed_kernel(const uint32_t *__restrict__ params, uint32_t *__restrict__ states,
            uint32_t stride, uint32_t n_streams) {
    // rows padded by one word: the chain lanes write one column
    __shared__ uint32_t tile[SEED_STREAMS][SEED_TILE + 1];
    const uint32_t lane = threadIdx.x, k0 = blockIdx.x * SEED_STREAMS;
    const uint32_t rows = n_streams - k0 < SEED_STREAMS ? n_streams - k0 : SEED_STREAMS;
    const uint32_t n = params[(uint64_t)k0 * P_WORDS + P_N];  // one exponent per set
    uint32_t x = lane < rows ? params[(uint64_t)(k0 + lane) * P_WORDS + P_SEED] : 0u;
    gptr<uint32_t> s = (gptr<uint32_t>)(states + (uint64_t)k0 * stride);
    for (uint32_t i0 = 0; i0 < n; i0 += SEED_TILE) {
        if (lane < SEED_STREAMS) {
            // x holds word i0; the words past n are never stored
#pragma unroll 16
            for (uint32_t j = 0; j < SEED_TILE; ++j) {
                tile[lane][j] = x;
                x = 1812433253u * (x ^ (x >> 30)) + (i0 + j + 1u);
            }
        }
        group_sync<64>();
        const uint32_t i = i0 + lane;
        if (i < n)
            for (uint32_t r = 0; r < rows; ++r) s[(uint64_t)r * stride + i] = tile[r][lane];
        group_sync<64>();
    }
}

__global__ void reset_counter_kernel(uint32_t *counter) { *counter = 0u; }

__global__ void clear_kernel(uint32_t *p, uint32_t n) {
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0u;
}

// One wave; lane i owns header word i (i < 26).  Every lane reads the tag
// before any lane writes it.
__global__ void header_kernel(uint32_t *hdr, uint32_t tag_lo, uint32_t tag_hi,
                              uint32_t clear_errors) {
    const uint32_t i = threadIdx.x;
    const bool fresh = hdr[HDR_TAG] != tag_lo || hdr[HDR_TAG + 1] != tag_hi;
    __builtin_amdgcn_wave_barrier();
    const bool claim = i < (uint32_t)HDR_ERR || i == (uint32_t)HDR_J_CLAIM ||
                       i == (uint32_t)HDR_W_CLAIM || i == (uint32_t)HDR_B_CLAIM;
    const bool errw = i >= (uint32_t)HDR_ERR && i < (uint32_t)(HDR_ERR + HDR_ERR_WORDS);
    const bool stamp = i >= HDR_STAMP_BYTE / 4 && i < HDR_STAMP_BYTE / 4 + 8;
    if (claim || (errw && (fresh || clear_errors)) || (stamp && fresh)) hdr[i] = 0u;
    if (i == (uint32_t)HDR_TAG) hdr[i] = tag_lo;
    if (i == (uint32_t)HDR_TAG + 1) hdr[i] = tag_hi;
}

// Device timestamp (the constant-rate wall clock) for phase timing.
__global__ void stamp_kernel(uint64_t *dst) {
    if (threadIdx.x == 0) *dst = wall_clock64();
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Store-only fill: the achievable write bandwidth next to the generator
// (plain stores, as the generator uses; on gfx950 they measured faster than
// non-temporal ones).
__global__ void __launch_bounds__(256)
fill_kernel(u32x4 *__restrict__ out, uint64_t n_vec, uint32_t *__restrict__ tail,
            uint32_t n_tail, uint32_t value) {
    const u32x4 v = {value, value, value, value};
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_vec; i += stride)
        out[i] = v;
    if (blockIdx.x == 0 && threadIdx.x < n_tail) tail[threadIdx.x] = value;
}

// Copies a list of pieces, one workgroup each, by the widest unit that source,
// destination and size allow.  Results that come back together leave in one
// launch: a copy command each costs the caller about 5 us, more than the
// bytes of a short result (1000 requests, 0.5 GB: 3.9 ms against 6.0).
template <typename T>
__device__ __forceinline__ void copy_units(const CopyPiece &c) {
    gptr<const T> src = (gptr<const T>)(reinterpret_cast<const T *>(c.src));
    gptr<T> dst = (gptr<T>)(reinterpret_cast<T *>(c.dst));
    const uint32_t n = (uint32_t)(c.bytes / sizeof(T));
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) dst[i] = src[i];
}

__global__ void __launch_bounds__(256)
copy_kernel(const CopyPiece *__restrict__ pieces) {
    const CopyPiece c = pieces[blockIdx.x];
    const uint64_t all = c.src | c.dst | c.bytes;
    if ((all & 15u) == 0) copy_units<u32x4>(c);
    else if ((all & 3u) == 0) copy_units<uint32_t>(c);
    else copy_units<uint8_t>(c);
}

// ------------------------------------------------------------- dispatch --

typedef void (*GenFn)(const uint32_t *, const BatchItem *, uint32_t, uint32_t *, uint32_t,
                      uint32_t, PlainArgs);

// Launches one of the generation kernels with the LDS of Core<N, TPS, K>
// times the groups per workgroup; persistent launches fill every CU to its
// occupancy with no more groups than items.
template <int N, int TPS, int K, int WPB, bool GRP = false>
static hipError_t launch_with(GenFn fn, bool *attr_set, const LaunchArgs &a) {
    using C = Core<N, TPS, K, GRP>;
    const int threads = TPS == 64 ? 64 * WPB : TPS;
    const size_t lds = (size_t)C::LDS_WORDS * 4 * (TPS == 64 ? WPB : 1);
    if (!*attr_set) {  // benign race: idempotent attribute
        hipError_t e = hipFuncSetAttribute((const void *)fn,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds);
        if (e != hipSuccess) return e;
        *attr_set = true;
    }
    const int per_block = TPS == 64 ? WPB : 1;
    const int need = (int)((a.n_items + per_block - 1) / per_block);
    int grid = need > 0 ? need : 1;
    if (a.persistent) {
        int per_cu = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds);
        if (e != hipSuccess) return e;
        if (a.groups_per_cu > 0 && a.groups_per_cu < per_cu) per_cu = a.groups_per_cu;
        if (per_cu < 1) per_cu = 1;
        if (per_cu * a.num_cus < grid) grid = per_cu * a.num_cus;
    }
    PlainArgs plain{a.plain_states, a.plain_stride, a.plain_mode, a.plain_out, a.plain_count};
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(fn, dim3(grid), dim3(threads), lds, (hipStream_t)a.stream, a.params,
                       a.items, a.n_items, a.counter, a.persistent ? 1u : 0u, a.win_below, plain);
    return hipGetLastError();
}

template <int N, int TPS, int K, int WPB, bool GRP>
static hipError_t launch_gen(const LaunchArgs &a) {
    static bool attr_set = false;
    return launch_with<N, TPS, K, WPB, GRP>(gen_kernel<N, TPS, K, WPB, GRP>, &attr_set, a);
}

template <int N>
static hipError_t launch_prefix_n(const LaunchArgs &a) {
    static bool attr_set = false;
    return launch_with<N, 64, prefix_k(N), 4>(prefix_kernel<N>, &attr_set, a);
}

template <int N>
static hipError_t launch_check_n(const LaunchArgs &a) {
    constexpr int lds = Core<N, 64, 1>::LDS_WORDS * 4 * 4;
    static bool attr_set = false;  // benign race: idempotent attribute
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)check_kernel<N>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    // one request per wave up to two waves per SIMD, so that requests which
    // do have to be regenerated run beside one another
    const uint32_t waves = (uint32_t)(a.num_cus > 0 ? a.num_cus : 1) * 8u;
    uint32_t per_wave = (a.n_items + waves - 1) / waves;
    if (per_wave > 64u) per_wave = 64u;
    if (per_wave < 1u) per_wave = 1u;
    const uint32_t grid = (a.n_items + 4 * per_wave - 1) / (4 * per_wave);
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(check_kernel<N>, dim3(grid > 0 ? grid : 1), dim3(256), lds,
                       (hipStream_t)a.stream, a.params, a.items, a.n_items, per_wave, a.err,
                       a.win_below);
    return hipGetLastError();
}

template <int N>
static hipError_t launch_sparse_n(const LaunchArgs &a, uint32_t n_wide, uint32_t *wide_counter) {
    constexpr int lds = sparse_lds_words<N>() * 4;
    static bool attr_set = false;  // benign race: idempotent attribute
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)sparse_kernel<N>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    uint32_t grid = n_wide + (a.n_items - n_wide + 3) / 4;
    const uint32_t cap = (uint32_t)a.num_cus * (uint32_t)(160 * 1024 / lds);
    if (grid > cap) grid = cap;
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(sparse_kernel<N>, dim3(grid > 0 ? grid : 1), dim3(256), lds,
                       (hipStream_t)a.stream, a.params, a.items, n_wide, a.n_items, wide_counter,
                       a.counter, a.win_below);
    return hipGetLastError();
}

hipError_t launch_sparse(int n_words, const LaunchArgs &a, uint32_t n_wide,
                         uint32_t *wide_counter) {
    switch (n_words) {
        case 351: return launch_sparse_n<351>(a, n_wide, wide_counter);
        case 726: return launch_sparse_n<726>(a, n_wide, wide_counter);
        case 1391: return launch_sparse_n<1391>(a, n_wide, wide_counter);
        default: return hipErrorInvalidValue;
    }
}

template <int N>
static hipError_t launch_few_n(const LaunchArgs &a) {
    static bool attr_set = false;
    return launch_with<N, 64, 8, 4>(few_kernel<N>, &attr_set, a);
}

hipError_t launch_few(int n_words, const LaunchArgs &a) {
    switch (n_words) {
        case 101: return launch_few_n<101>(a);
        case 351: return launch_few_n<351>(a);
        case 726: return launch_few_n<726>(a);
        case 1391: return launch_few_n<1391>(a);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_prefix(int n_words, const LaunchArgs &a) {
    switch (n_words) {
        case 101: return launch_prefix_n<101>(a);
        case 351: return launch_prefix_n<351>(a);
        case 726: return launch_prefix_n<726>(a);
        case 1391: return launch_prefix_n<1391>(a);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_check(int n_words, const LaunchArgs &a) {
    switch (n_words) {
        case 101: return launch_check_n<101>(a);
        case 351: return launch_check_n<351>(a);
        case 726: return launch_check_n<726>(a);
        case 1391: return launch_check_n<1391>(a);
        default: return hipErrorInvalidValue;
    }
}

template <int N, int TPS, int K, int WPB, bool GRP>
static size_t lds_bytes_of() {
    return (size_t)Core<N, TPS, K, GRP>::LDS_WORDS * 4 * (TPS == 64 ? WPB : 1);
}

// Streams a CU runs at once with this variant (waves for TPS = 64, else
// workgroups), from the occupancy the runtime reports; 0 on error.
template <int N, int TPS, int K, int WPB, bool GRP>
static int slots_of() {
    static int cached = -1;  // benign race: idempotent query
    if (cached < 0) {
        int per_cu = 0;
        const int threads = TPS == 64 ? 64 * WPB : TPS;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &per_cu, gen_kernel<N, TPS, K, WPB, GRP>, threads,
                lds_bytes_of<N, TPS, K, WPB, GRP>()) != hipSuccess)
            return 0;
        cached = per_cu * (TPS == 64 ? WPB : 1);
    }
    return cached;
}

// A launch variant: [0] without groups, [1] with (the same where there are
// none).
struct Variant {
    int N, tps, k, wpb;
    hipError_t (*launch[2])(const LaunchArgs &);
    size_t (*lds[2])();
    int (*slots[2])();
};

#define MTGP_G(N, T) ((T) == 64 && has_groups(N))
#define MTGP_V(N, T, K, P)                                                              \
    {N, T, K, P,                                                                        \
     {&launch_gen<N, T, K, P, false>, &launch_gen<N, T, K, P, MTGP_G(N, T)>},           \
     {&lds_bytes_of<N, T, K, P, false>, &lds_bytes_of<N, T, K, P, MTGP_G(N, T)>},       \
     {&slots_of<N, T, K, P, false>, &slots_of<N, T, K, P, MTGP_G(N, T)>}}
#define MTGP_VARIANTS(N)                                                              \
    MTGP_V(N, 64, 1, 4), MTGP_V(N, 64, 2, 4), MTGP_V(N, 64, 4, 4), MTGP_V(N, 64, 8, 4), \
    MTGP_V(N, 64, 2, 8), MTGP_V(N, 64, 4, 8), MTGP_V(N, 64, 4, 16),                   \
    MTGP_V(N, 256, 1, 1), MTGP_V(N, 256, 2, 1), MTGP_V(N, 512, 1, 1),                 \
    MTGP_V(N, 512, 2, 1), MTGP_V(N, 1024, 1, 1)

static const Variant kVariants[] = {
    MTGP_VARIANTS(101), MTGP_VARIANTS(351), MTGP_VARIANTS(726), MTGP_VARIANTS(1391),
};

// LDS per workgroup on gfx950.
static constexpr size_t kLdsBytes = 160 * 1024;

static bool fits(const Variant &v) { return v.lds[1]() + 64 <= kLdsBytes; }

int variant_count(int n_words, VariantInfo *out, int max_out) {
    int c = 0;
    for (const Variant &v : kVariants) {
        if (v.N != n_words || !fits(v)) continue;
        if (out && c < max_out) {
            out[c].tps = v.tps;
            out[c].k = v.k;
            out[c].wpb = v.wpb;
            for (int g = 0; g < 2; ++g) out[c].lds_bytes[g] = v.lds[g]();
        }
        ++c;
    }
    return c;
}

hipError_t launch_variant(int n_words, int tps, int k, int wpb, const LaunchArgs &a,
                          bool *found) {
    for (const Variant &v : kVariants) {
        if (v.N == n_words && v.tps == tps && v.k == k && v.wpb == wpb && fits(v)) {
            *found = true;
            return v.launch[a.groups ? 1 : 0](a);
        }
    }
    *found = false;
    return hipSuccess;
}

int variant_slots_per_cu(int n_words, int tps, int k, int wpb, bool groups) {
    for (const Variant &v : kVariants)
        if (v.N == n_words && v.tps == tps && v.k == k && v.wpb == wpb && fits(v))
            return v.slots[groups ? 1 : 0]();
    return 0;
}

template <int T>
static hipError_t launch_jump_t(const JumpBlock *blocks, uint32_t n_blocks, int num_cus,
                                hipStream_t s) {
    constexpr int lds = jump_lds_words(T) * 4;
    static bool attr_set = false;  // benign race: idempotent attribute
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)jump_kernel<T>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    int grid = (int)n_blocks;
    const int cap = num_cus * (160 * 1024 / lds);  // workgroups that fit the CUs' LDS
    if (grid > cap) grid = cap;
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(jump_kernel<T>, dim3(grid), dim3(64 * JUMP_WAVES), lds, s, blocks,
                       n_blocks);
    return hipGetLastError();
}

hipError_t launch_jump(int n_words, const JumpBlock *blocks, uint32_t n_blocks, int num_cus,
                       hipStream_t s) {
    if (n_blocks == 0) return hipSuccess;
    switch (n_words) {
        case 101: return launch_jump_t<jump_tiles(101)>(blocks, n_blocks, num_cus, s);
        case 351: return launch_jump_t<jump_tiles(351)>(blocks, n_blocks, num_cus, s);
        case 726: return launch_jump_t<jump_tiles(726)>(blocks, n_blocks, num_cus, s);
        case 1391: return launch_jump_t<jump_tiles(1391)>(blocks, n_blocks, num_cus, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_seed(const uint32_t *params, uint32_t *states, uint32_t stride,
                       uint32_t n_streams, hipStream_t s) {
    const int grid = (int)((n_streams + SEED_STREAMS - 1) / SEED_STREAMS);
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(seed_kernel, dim3(grid), dim3(64), 0, s, params, states, stride,
                       n_streams);
    return hipGetLastError();
}

hipError_t launch_reset(uint32_t *counter, hipStream_t s) {
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(1), 0, s, counter);
    return hipGetLastError();
}

hipError_t launch_clear(uint32_t *p, uint32_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(clear_kernel, dim3(1), dim3(64), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_header(uint32_t *hdr, uint64_t tag, bool clear_errors, hipStream_t s) {
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(header_kernel, dim3(1), dim3(64), 0, s, hdr, (uint32_t)tag,
                       (uint32_t)(tag >> 32), clear_errors ? 1u : 0u);
    return hipGetLastError();
}

hipError_t launch_stamp(uint64_t *dst, hipStream_t s) {
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(stamp_kernel, dim3(1), dim3(64), 0, s, dst);
    return hipGetLastError();
}

// The device API reads the same parameter blocks the library writes.
static_assert(MTGP_DP_N == P_N && MTGP_DP_POS == P_POS && MTGP_DP_SH1 == P_SH1 &&
                  MTGP_DP_SH2 == P_SH2 && MTGP_DP_MASK == P_MASK && MTGP_DP_REC == P_REC &&
                  MTGP_DP_TMP == P_TMP && MTGP_DP_FLT == P_FLT && MTGP_DP_WORDS == P_WORDS &&
                  MTGP_DP_WIN_WN == P_WIN_WN && MTGP_DP_WIN_E == P_WIN_E &&
                  MTGP_DP_WIN_Q == P_WIN_Q && MTGP_DP_WIN_MAT == P_WIN_MAT &&
                  MTGP_DEVICE_WIN_E == WIN_EMAX &&
                  MTGP_DEVICE_WIN_MATS == WIN_MAXROUNDS * WIN_MAT_WORDS,
              "device API parameter layout");

// Generation through the device-side draw API: workgroup k owns stream k and
// writes count outputs at out + k*count, drawing blockDim.x at a time.
template <bool F32>
__global__ void __launch_bounds__(1024)
workgroup_kernel(const uint32_t *__restrict__ params, uint32_t *__restrict__ states,
                 uint32_t stride, uint64_t count, uint32_t *__restrict__ out,
                 uint32_t lds_words) {
    extern __shared__ uint32_t lds[];
    mtgp_device_stream s;
    const uint32_t k = blockIdx.x;
    uint32_t *row = states + (uint64_t)k * stride;
    mtgp_device_begin(s, params, k, row, lds, lds_words);
    gptr<uint32_t> o = (gptr<uint32_t>)(out + (uint64_t)k * count);
    for (uint64_t done = 0; done < count; done += blockDim.x) {
        const uint64_t rem = count - done;
        const uint32_t n = rem < blockDim.x ? (uint32_t)rem : blockDim.x;
        const uint32_t r = mtgp_device_draw_bits<F32>(s, n);
        if (threadIdx.x < n) o[done + threadIdx.x] = r;
    }
    mtgp_device_end(s, row);
}

hipError_t launch_workgroup(const uint32_t *params, uint32_t *states, uint32_t stride,
                            uint32_t n_streams, uint64_t count, uint32_t *out, uint32_t f32,
                            uint32_t threads, uint32_t n_words, hipStream_t s) {
    const uint32_t words = MTGP_DEVICE_LDS_WORDS(n_words, threads);
    auto fn = f32 ? workgroup_kernel<true> : workgroup_kernel<false>;
    static bool attr_set[2] = {false, false};  // benign race: idempotent attribute
    if (!attr_set[f32 ? 1 : 0]) {
        hipError_t e = hipFuncSetAttribute((const void *)fn,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)MTGP_DEVICE_LDS_WORDS(1391u, 1024u) * 4);
        if (e != hipSuccess) return e;
        attr_set[f32 ? 1 : 0] = true;
    }
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(fn, dim3(n_streams), dim3(threads), (size_t)words * 4, s, params, states,
                       stride, count, out, words);
    return hipGetLastError();
}

// Screening statistics over generated uint32 outputs, one workgroup per
// stream of `count` words at out + k*count:
//  gap test (Knuth, Sec. 3.3.2 D, between consecutive hits): a hit is a word
//    in [lo, hi); the gap between consecutive hits j < j' is j' - j - 1,
//    counted in bin min(gap, bins-1);
//  Hamming-weight dependency: the weight class of a word (popcount <= 14,
//    15..17, >= 18) and of its successor, counted in a 3x3 table.
// counts[k * (bins + 9) ..] = gap bins, then the table row-major.
// Wave w takes the region [w R, (w+1) R) of the stream (R a multiple of 32)
// in tiles of 2048 words: 16-byte loads of consecutive words, the next
// tile's in flight while this one is counted, turned in LDS so that a lane
// holds 32 consecutive words.  Per word a lane only shifts three bits into
// registers: class 0 (the sign of popcount - 15), class 2 (the sign of
// 17 - popcount) and the hit.  All counting is then popcounts of 32-word
// masks against themselves moved by one word (weight pairs) or by d words
// (gaps of d - 1); the previous 32 words are the lane below's.  Gaps that
// SCREEN_D rounds leave open are counted one hit at a time.  Of the weight
// table only the four corners and the two classes' totals are counted; the
// class-1 entries follow from the sums.  Gaps across regions are added at
// the end, in region order.  Bound by its reads: 4000 streams x 2^17 words,
// one word in four a hit, 363 us, 5.8 TB/s (a hit ballot per 64-word slice
// and a pair counter per word: 727 us, bound by vector work).
constexpr uint32_t SCREEN_NONE = 0xFFFFFFFFu;  // no hit yet (positions < count < 2^32)
constexpr uint32_t SCREEN_TILE = 2048;
constexpr uint32_t SCREEN_ROW = 36;            // LDS words per lane: 32, padded

// 16-byte loads at any word address (a stream starts at k * count words).
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Sum over the wave's lanes, for every lane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += (uint32_t)__shfl_xor((int)v, d, 64);
    return v;
}

template <int NW, int D0>
__global__ void __launch_bounds__(64 * NW)
screen_kernel(const uint32_t *__restrict__ out, uint64_t count, uint32_t lo, uint32_t hi,
              uint32_t bins, uint64_t *__restrict__ counts) {
    __shared__ u32x4 turn[NW][64 * SCREEN_ROW / 4];
    __shared__ uint32_t hist[64 + 9];
    __shared__ uint32_t first_hit[NW], last_hit[NW];
    const uint32_t k = blockIdx.x, tid = threadIdx.x;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63u;
    for (uint32_t i = tid; i < bins + 9; i += 64 * NW) hist[i] = 0;
    __syncthreads();
    gptr<const uint32_t> x = (gptr<const uint32_t>)(out + (uint64_t)k * count);
    const uint32_t n = (uint32_t)count;
    const uint32_t R = (uint32_t)((count + 32 * NW - 1) / (32 * NW) * 32);
    const uint32_t r0 = (uint64_t)wave * R < n ? wave * R : n;
    const uint32_t r1 = n - r0 < R ? n : r0 + R;
    const uint32_t span = hi - lo;  // a hit: v - lo < span
    const uint64_t lanes_below = lane ? ~0ull >> (64u - lane) : 0ull;
    uint32_t first = SCREEN_NONE, carry = SCREEN_NONE;  // region's first and last hit so far
    uint32_t carry_h = 0, carry_z = 0, carry_t = 0;     // masks of the 32 words before the tile
    if (r0 > 0 && r0 < r1) {  // the word before the region: the first pair's left class
        const int w = __builtin_popcount(x[r0 - 1]);
        carry_z = w <= 14 ? 1u : 0u;
        carry_t = w >= 18 ? 1u : 0u;
    }
    uint32_t n00 = 0, n02 = 0, n20 = 0, n22 = 0, c0 = 0, c2 = 0, p0 = 0, p2 = 0;
    uint32_t gap[D0 > 0 ? D0 : 1];
#pragma unroll
    for (int d = 0; d < D0; ++d) gap[d] = 0;
    u32x4 v[8];
    auto load = [&](uint32_t b) {  // words b + 256 q + 4 lane ..., zeros past the region
        if (r1 - b >= SCREEN_TILE) {
            gptr<const u32x4u> p = (gptr<const u32x4u>)(x + b + 4 * lane);
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = p[64 * q];
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t j = b + 256u * q + 4u * lane + e;
                    v[q][e] = j < r1 ? x[j] : 0u;
                }
        }
    };
    if (r0 < r1) load(r0);
    for (uint32_t b = r0; b < r1;) {
        u32x4 *row = turn[wave];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            row[(8 * q + (lane >> 3)) * (SCREEN_ROW / 4) + (lane & 7u)] = v[q];
        group_sync<64>();
        u32x4 t[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) t[q] = row[lane * (SCREEN_ROW / 4) + q];
        group_sync<64>();
        const uint32_t mine = b + 32u * lane;  // this lane's first word
        const uint32_t left = r1 - b > 32u * lane ? r1 - b - 32u * lane : 0u;
        b = r1 - b > SCREEN_TILE ? b + SCREEN_TILE : r1;
        if (b < r1) load(b);
        uint32_t Z = 0, T = 0, H = 0;  // first word in bit 31
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t w = t[q][e];
                const uint32_t low = (uint32_t)__builtin_popcount(w) - 15u;
                Z = __builtin_amdgcn_alignbit(Z, low, 31);
                T = __builtin_amdgcn_alignbit(T, 2u - low, 31);
                H = H + H + (w - lo < span ? 1u : 0u);
            }
        const uint32_t valid = left >= 32u ? ~0u : ~(~0u >> left);
        Z &= valid;
        T &= valid;
        H &= valid;
        uint32_t zp = (uint32_t)__shfl_up((int)Z, 1, 64), tp = (uint32_t)__shfl_up((int)T, 1, 64),
                 hp = (uint32_t)__shfl_up((int)H, 1, 64);
        if (lane == 0) {
            zp = carry_z;
            tp = carry_t;
            hp = carry_h;
        }
        carry_z = (uint32_t)__builtin_amdgcn_readlane((int)Z, 63);
        carry_t = (uint32_t)__builtin_amdgcn_readlane((int)T, 63);
        carry_h = (uint32_t)__builtin_amdgcn_readlane((int)H, 63);
        // left classes of the pairs that end at this lane's words
        const uint32_t zl = __builtin_amdgcn_alignbit(zp, Z, 1) & valid;
        const uint32_t tl = __builtin_amdgcn_alignbit(tp, T, 1) & valid;
        n00 += (uint32_t)__builtin_popcount(zl & Z);
        n02 += (uint32_t)__builtin_popcount(zl & T);
        n20 += (uint32_t)__builtin_popcount(tl & Z);
        n22 += (uint32_t)__builtin_popcount(tl & T);
        c0 += (uint32_t)__builtin_popcount(Z);
        c2 += (uint32_t)__builtin_popcount(T);
        p0 += (uint32_t)__builtin_popcount(zl);
        p2 += (uint32_t)__builtin_popcount(tl);
        // hits whose previous hit lies d words before them, d = 1 .. D0
        uint32_t open = H;
#pragma unroll
        for (int d = 1; d <= D0; ++d) {
            const uint32_t hd = __builtin_amdgcn_alignbit(hp, H, d);
            gap[d - 1] += (uint32_t)__builtin_popcount(open & hd);
            open &= ~hd;
        }
        const uint64_t any = __builtin_amdgcn_ballot_w64(H != 0u);
        if (any) {
            const uint32_t last = mine + 31u - (uint32_t)__builtin_ctz(H | 0x80000000u);
            if (__builtin_amdgcn_ballot_w64(open != 0u)) {
                // the last hit before this lane's words
                const uint64_t below = any & lanes_below;
                const uint32_t from =
                    (uint32_t)__shfl((int)last, below ? 63 - __builtin_clzll(below) : 0, 64);
                const uint32_t before = below ? from : carry;
                while (open) {
                    const uint32_t i = (uint32_t)__builtin_clz(open);  // word mine + i
                    open &= ~(0x80000000u >> i);
                    const uint32_t earlier = i ? H >> (32u - i) : 0u;
                    const uint32_t prev =
                        earlier ? mine + i - 1u - (uint32_t)__builtin_ctz(earlier) : before;
                    if (prev != SCREEN_NONE) {
                        const uint32_t g = mine + i - prev - 1u;
                        atomicAdd(&hist[g < bins - 1u ? g : bins - 1u], 1u);
                    }
                }
            }
            if (first == SCREEN_NONE) {
                const int at = __builtin_ctzll(any);
                first = (uint32_t)__builtin_amdgcn_readlane(
                    (int)(mine + (uint32_t)__builtin_clz(H | 1u)), at);
            }
            carry = (uint32_t)__builtin_amdgcn_readlane((int)last, 63 - __builtin_clzll(any));
        }
    }
    if (r0 < r1) {
#pragma unroll
        for (int d = 0; d < D0; ++d) {
            const uint32_t g = wave_sum(gap[d]);
            if (lane == 0 && g)
                atomicAdd(&hist[(uint32_t)d < bins - 1u ? (uint32_t)d : bins - 1u], g);
        }
        n00 = wave_sum(n00);
        n02 = wave_sum(n02);
        n20 = wave_sum(n20);
        n22 = wave_sum(n22);
        c0 = wave_sum(c0);
        c2 = wave_sum(c2);
        p0 = wave_sum(p0);
        p2 = wave_sum(p2);
        uint32_t pairs = r1 - r0;
        if (r0 == 0) {  // the stream's first word ends no pair
            const int w = __builtin_popcount(x[0]);
            --pairs;
            c0 -= w <= 14 ? 1u : 0u;
            c2 -= w >= 18 ? 1u : 0u;
        }
        if (lane == 0) {
            const uint32_t n01 = p0 - n00 - n02, n21 = p2 - n20 - n22;
            const uint32_t n10 = c0 - n00 - n20, n12 = c2 - n02 - n22;
            const uint32_t tab[9] = {n00, n01, n02, n10, pairs - p0 - p2 - n10 - n12, n12,
                                     n20, n21, n22};
#pragma unroll
            for (int q = 0; q < 9; ++q) atomicAdd(&hist[bins + q], tab[q]);
        }
    }
    if (lane == 0) {
        first_hit[wave] = first;
        last_hit[wave] = carry;
    }
    __syncthreads();
    if (tid == 0) {
        // gaps across regions, in region order
        uint32_t pl = SCREEN_NONE;
        for (int w = 0; w < NW; ++w) {
            if (first_hit[w] == SCREEN_NONE) continue;
            if (pl != SCREEN_NONE) {
                const uint32_t g = first_hit[w] - pl - 1u;
                hist[g < bins - 1u ? g : bins - 1u] += 1u;
            }
            pl = last_hit[w];
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < bins + 9; i += 64 * NW)
        counts[(uint64_t)k * (bins + 9) + i] = hist[i];
}

template <int NW>
static void launch_screen_n(const uint32_t *out, uint32_t n_streams, uint64_t count, uint32_t lo,
                            uint32_t hi, uint32_t bins, uint64_t *counts, hipStream_t s) {
    // Rounds of whole-mask gap counting (four operations per 32 words each)
    // against one loop turn per hit left open in the busiest lane: words
    // hit more often than 1 in 12 leave few hits after 16 rounds (1 in 2:
    // after 8), rarer hits are counted one at a time from the start.
    const uint32_t span = hi - lo;
    const dim3 grid(n_streams), block(64 * NW);
    if (span >= (1u << 30) + (1u << 29))
        hipLaunchKernelGGL((screen_kernel<NW, 8>), grid, block, 0, s, out, count, lo, hi, bins,
                           counts);
    else if (span >= (1u << 28) + (1u << 26))
        hipLaunchKernelGGL((screen_kernel<NW, 16>), grid, block, 0, s, out, count, lo, hi, bins,
                           counts);
    else
        hipLaunchKernelGGL((screen_kernel<NW, 0>), grid, block, 0, s, out, count, lo, hi, bins,
                           counts);
}

hipError_t launch_screen(const uint32_t *out, uint32_t n_streams, uint64_t count, uint32_t lo,
                         uint32_t hi, uint32_t bins, uint64_t *counts, hipStream_t s) {
    (void)hipGetLastError();  // report this launch only
    // Waves per stream: one where a stream is at most two tiles, 16 where
    // fewer than two workgroups per CU would run (streams are not shared
    // between workgroups), else four.
    if (count <= 2 * SCREEN_TILE)
        launch_screen_n<1>(out, n_streams, count, lo, hi, bins, counts, s);
    else if (n_streams < 512 && count > 16 * SCREEN_TILE)
        launch_screen_n<16>(out, n_streams, count, lo, hi, bins, counts, s);
    else
        launch_screen_n<4>(out, n_streams, count, lo, hi, bins, counts, s);
    return hipGetLastError();
}

hipError_t launch_copy(const CopyPiece *pieces, uint32_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(copy_kernel, dim3(n), dim3(256), 0, s, pieces);
    return hipGetLastError();
}

hipError_t launch_fill(uint32_t *out, uint64_t n_words, uint32_t value, int num_cus,
                       hipStream_t s) {
    const uint64_t n_vec = n_words / 4;
    const uint32_t n_tail = (uint32_t)(n_words % 4);
    uint64_t want = (n_vec + 255) / 256;
    uint64_t cap = (uint64_t)num_cus * 8;
    int grid = (int)(want < cap ? (want > 0 ? want : 1) : cap);
    (void)hipGetLastError();  // report this launch only
    hipLaunchKernelGGL(fill_kernel, dim3(grid), dim3(256), 0, s,
                       reinterpret_cast<u32x4 *>(out), n_vec, out + n_vec * 4, n_tail, value);
    return hipGetLastError();
}

}  // namespace mtgp
