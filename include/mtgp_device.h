/*
 * mtgp_device.h -- device-side draw API: a workgroup of a user kernel owns
 * one stream and draws from it with its state kept in LDS, without an HBM
 * round trip per number.
 *
 * This is the paper's consumer model made explicit (Sec. 2, Sec. 3.2): the
 * generator belongs to one thread block, its state is manipulated in the
 * block's shared memory, and it persists in device memory between kernel
 * calls.  The numbers are exactly those of mtgp_generate_u32/f32 (the same
 * definition, see mtgp.h), in the same order: a stream advances by the
 * number of outputs drawn, whatever the dtype and however the draws are cut.
 *
 * Use (all threads of the workgroup call every function, uniformly):
 *
 *     extern __shared__ uint32_t lds[];           // MTGP_DEVICE_LDS_WORDS(N, T)
 *     mtgp_device_stream s;
 *     mtgp_device_begin(s, d_params, k, d_states + k * stride, lds, words);
 *     uint32_t r = mtgp_device_draw_u32(s, n);    // thread t < n gets output t
 *     float f = mtgp_device_draw_f32(s, n);
 *     mtgp_device_end(s, d_states + k * stride);
 *
 * d_params is the parameter buffer written by mtgp_init_states (its layout
 * is given below), d_states a state row of N words.  The workgroup is
 * one-dimensional with T = blockDim.x threads (a multiple of 64, at most
 * 1024); a draw produces n <= T outputs in steps of at most W = N - pos
 * words, so streams with a small step width take several steps per draw.
 * Concurrent use of one stream by two workgroups is a race.
 */
#ifndef MTGP_DEVICE_H
#define MTGP_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

/* Word offsets in a stream's device parameter block (MTGP_DP_WORDS words per
 * stream, stream k at d_params + k * MTGP_DP_WORDS). */
enum : uint32_t {
    MTGP_DP_MEXP = 0,
    MTGP_DP_N = 1,     /* state words */
    MTGP_DP_POS = 2,
    MTGP_DP_SH1 = 3,
    MTGP_DP_SH2 = 4,
    MTGP_DP_MASK = 5,
    MTGP_DP_REC = 16,  /* rec_tbl[16], then tmp_tbl[16] at 32, flt_tbl[16] at 48 */
    MTGP_DP_TMP = 32,
    MTGP_DP_FLT = 48,
    /* streams with W < 64 and a GF(2)-linear rec_tbl (else all zero): */
    MTGP_DP_WIN_WN = 64,     /* words of a window, at most N - 1 */
    MTGP_DP_WIN_E = 65,      /* elements per lane and window */
    MTGP_DP_WIN_Q = 66,      /* lanes per residue class mod W */
    MTGP_DP_WIN_MAT = 128,   /* nibble tables of M^(E*2^k), 128 words each */
    MTGP_DP_WORDS = 1024,
};
enum : uint32_t { MTGP_DEVICE_WIN_E = 8, MTGP_DEVICE_WIN_MATS = 640 };
/* A window takes as long as about 16 dependent steps of W words (1.8 us
 * against 105 ns a step, mexp 11213): draws of fewer steps take the steps. */
enum : uint32_t { MTGP_DEVICE_WIN_STEPS = 16 };

/* LDS words a workgroup of T threads needs for a stream of N state words:
 * a buffer of 2N + 4T words (compacted, without overlap, when full), the
 * three tables and the window's matrices.  2N + 4T + 48 words are enough to
 * run; the window of narrow streams then is not used. */
#define MTGP_DEVICE_LDS_WORDS(n_words, threads) \
    (2u * (n_words) + 4u * (threads) + 48u + MTGP_DEVICE_WIN_MATS)

struct mtgp_device_stream {
    uint32_t *buf;  /* LDS: state buffer, then rec, tmp, flt tables, matrices */
    uint32_t cap;   /* buffer words */
    uint32_t h;     /* buffer index of the next word */
    uint32_t N, W, sh1, sh2, mask;
    uint32_t lin;                    /* rec_tbl is known to be linear */
    uint32_t win_n, win_e;           /* window: words, elements per lane; win_e == 0: none */
    uint32_t win_r, win_sub;         /* this lane's residue class and chunk */
};

/* Loads stream `stream_id`'s tables and its state d_state[0..N) into lds
 * (lds_words >= MTGP_DEVICE_LDS_WORDS(N, blockDim.x)). */
__device__ inline void mtgp_device_begin(mtgp_device_stream &s, const uint32_t *d_params,
                                         uint32_t stream_id, const uint32_t *d_state,
                                         uint32_t *lds, uint32_t lds_words) {
    const uint32_t *p = d_params + (uint64_t)stream_id * MTGP_DP_WORDS;
    s.N = p[MTGP_DP_N];
    s.W = s.N - p[MTGP_DP_POS];
    s.sh1 = p[MTGP_DP_SH1];
    s.sh2 = p[MTGP_DP_SH2];
    s.mask = p[MTGP_DP_MASK];
    s.buf = lds;
    const bool room = lds_words >= MTGP_DEVICE_LDS_WORDS(s.N, blockDim.x);
    s.cap = lds_words - 48u - (room ? MTGP_DEVICE_WIN_MATS : 0u);
    s.h = s.N;
    s.lin = s.win_n = s.win_e = s.win_r = s.win_sub = 0;
    if (s.W < 64u) {
        s.lin = p[MTGP_DP_WIN_E];
        if (s.lin && room && blockDim.x > MTGP_DEVICE_WIN_STEPS * s.W) {
            const uint32_t q = p[MTGP_DP_WIN_Q];   /* lanes per class */
            s.win_n = p[MTGP_DP_WIN_WN];
            s.win_e = s.lin;
            s.win_r = (threadIdx.x & 63u) / q;
            s.win_sub = (threadIdx.x & 63u) - s.win_r * q;
            for (uint32_t i = threadIdx.x; i < MTGP_DEVICE_WIN_MATS; i += blockDim.x)
                lds[s.cap + 48u + i] = p[MTGP_DP_WIN_MAT + i];
        }
    }
    for (uint32_t i = threadIdx.x; i < s.N; i += blockDim.x) lds[i] = d_state[i];
    for (uint32_t i = threadIdx.x; i < 48u; i += blockDim.x) lds[s.cap + i] = p[MTGP_DP_REC + i];
    __syncthreads();
}

/* Orders the LDS accesses of one wave across a step without a workgroup
 * barrier (a wave's LDS operations complete in issue order). */
__device__ inline void mtgp_device_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

/* Basis of a linear rec_tbl, and Y ^ rec_tbl[Y & 15] from it: the basis words
 * that the low four bits of Y select, without an LDS round trip on the
 * dependent chain. */
struct mtgp_device_basis {
    uint32_t b0, b1, b2, b3;
};

__device__ inline mtgp_device_basis mtgp_device_load_basis(const mtgp_device_stream &s) {
    const uint32_t *rec = s.buf + s.cap;
    return mtgp_device_basis{rec[1], rec[2], rec[4], rec[8]};
}

__device__ inline uint32_t mtgp_device_rec_linear(const mtgp_device_basis &r, uint32_t Y) {
    /* 0x78: a ^ (b & c) */
    uint32_t a = __builtin_amdgcn_bitop3_b32(Y, (uint32_t)__builtin_amdgcn_sbfe((int)Y, 0, 1),
                                             r.b0, 0x78);
    a = __builtin_amdgcn_bitop3_b32(a, (uint32_t)__builtin_amdgcn_sbfe((int)Y, 1, 1), r.b1, 0x78);
    a = __builtin_amdgcn_bitop3_b32(a, (uint32_t)__builtin_amdgcn_sbfe((int)Y, 2, 1), r.b2, 0x78);
    return __builtin_amdgcn_bitop3_b32(a, (uint32_t)__builtin_amdgcn_sbfe((int)Y, 3, 1), r.b3,
                                       0x78);
}

/* The words buf[h .. h + n) of a stream with W < 64 and a linear rec_tbl, on
 * the first wave alone; n <= win_n <= N - 1, so every x_{k-N} and x_{k-N+1}
 * is there.  What remains is the chain x_k = G(X_k) ^ M x_{k-W} of each
 * residue class mod W, which is affine: a class is cut into win_q chunks of
 * win_e words, one lane each; every lane runs its chunk from a zero carry
 * (the first chunk of a class from its true one), a scan with M^(E*2^i)
 * gives each chunk its true carry, and the lane runs its chunk again. */
__device__ inline void mtgp_device_window(mtgp_device_stream &s, uint32_t h, uint32_t n) {
    uint32_t *buf = s.buf;
    const uint32_t *mat = s.buf + s.cap + 48u;
    const mtgp_device_basis rb = mtgp_device_load_basis(s);
    const uint32_t lane = threadIdx.x, W = s.W;
    /* opaque: kept across calls, the loops' conditions would take more scalar
     * registers than there are */
    uint32_t E = __builtin_amdgcn_readfirstlane(s.win_e);
    asm volatile("" : "+s"(E));
    const uint32_t o = s.win_r + W * (s.win_sub * E);     /* the lane's first word */
    const uint32_t m = s.win_r < W && o < n ? n - o : 0u; /* words from it on */
    /* W's multiples, too: kept, they leave seven waves per SIMD (2048
     * workgroups of 256 threads, mexp 23209, all W wide, 4,096 words 29.6 us
     * against 25.7) */
    uint32_t W1 = __builtin_amdgcn_readfirstlane(W);
    asm volatile("" : "+s"(W1));
    uint32_t X[MTGP_DEVICE_WIN_E];
#pragma unroll
    for (uint32_t j = 0; j < MTGP_DEVICE_WIN_E; ++j) {
        X[j] = 0;
        if (j < E) {
            const uint32_t i = W1 * j < m ? h + o + W1 * j - s.N : h - s.N;
            const uint32_t x = (buf[i] & s.mask) ^ buf[i + 1];
            X[j] = x ^ (x << s.sh1);
        }
    }
    uint32_t c = s.win_sub == 0 && s.win_r < W ? buf[h + s.win_r - W] : 0u;
    const uint32_t chunks = (n + W * E - 1) / (W * E);    /* per class, as far as n reaches */
    if (chunks > 1) {
        uint32_t u = c;
#pragma unroll
        for (uint32_t j = 0; j < MTGP_DEVICE_WIN_E; ++j)
            if (j < E) u = mtgp_device_rec_linear(rb, X[j] ^ (u >> s.sh2));
        for (uint32_t d = 1; d < chunks; d <<= 1, mat += 128) {
            const uint32_t w = (uint32_t)__shfl((int)u, (int)(s.win_sub >= d ? lane - d : lane), 64);
            uint32_t y = 0;
#pragma unroll
            for (uint32_t k = 0; k < 8; k += 2)
                y = __builtin_amdgcn_bitop3_b32(y, mat[k * 16 + ((w >> (4 * k)) & 15u)],
                                                mat[k * 16 + 16 + ((w >> (4 * k + 4)) & 15u)],
                                                0x96);
            if (s.win_sub >= d) u ^= y;
        }
        const uint32_t in = (uint32_t)__shfl((int)u, (int)(s.win_sub ? lane - 1 : lane), 64);
        if (s.win_sub) c = in;
    }
#pragma unroll
    for (uint32_t j = 0; j < MTGP_DEVICE_WIN_E; ++j)
        if (j < E) {
            c = mtgp_device_rec_linear(rb, X[j] ^ (c >> s.sh2));
            if (W1 * j < m) buf[h + o + W1 * j] = c;
        }
    mtgp_device_wave_sync();
}

/* The same words in steps of W, on the first wave: lane l < W makes a step's
 * word l, whose pos tap is the word it made in the step before.  Four steps
 * at a time where the other two words of all four are there before (4W < N):
 * their LDS reads are then in flight together, and only the chain of the
 * lane's own words takes time. */
template <bool LIN>
__device__ inline void mtgp_device_steps(mtgp_device_stream &s, uint32_t h0, uint32_t n) {
    const uint32_t *tbl = s.buf + s.cap;
    const mtgp_device_basis rb = mtgp_device_load_basis(s);
    const uint32_t tid = threadIdx.x, sh1 = s.sh1, sh2 = s.sh2, mask = s.mask;
    /* opaque: as in mtgp_device_window */
    uint32_t W = __builtin_amdgcn_readfirstlane(s.W), N = __builtin_amdgcn_readfirstlane(s.N);
    asm volatile("" : "+s"(W), "+s"(N));
    if (tid < W) {
        uint32_t *p = s.buf + h0 + tid;
        uint32_t c = *(p - W), o = 0;
        if (4u * W < N)
            for (; o + 4u * W <= n; o += 4u * W, p += 4u * W) {
                uint32_t X[4];
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) {
                    const uint32_t *q = p + j * W - N;
                    X[j] = (q[0] & mask) ^ q[1];
                    X[j] ^= X[j] << sh1;
                }
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) {
                    const uint32_t Y = X[j] ^ (c >> sh2);
                    c = LIN ? mtgp_device_rec_linear(rb, Y) : Y ^ tbl[Y & 15u];
                    p[j * W] = c;
                }
                mtgp_device_wave_sync();
            }
        for (; o < n; o += W, p += W) {
            const uint32_t *q = p - N;
            uint32_t X = (q[0] & mask) ^ q[1];
            X ^= X << sh1;
            const uint32_t Y = X ^ (c >> sh2);
            c = LIN ? mtgp_device_rec_linear(rb, Y) : Y ^ tbl[Y & 15u];
            if (o + tid < n) *p = c;
            mtgp_device_wave_sync();
        }
    }
    mtgp_device_wave_sync();
}

/* Next n (<= blockDim.x) outputs: thread t < n receives output t as raw
 * bits (uint32 output, or the float32 output's bit pattern when F32).
 * The new state words are produced first, in steps of at most W words (a
 * word's recursion reads words at least W older); streams with W < 64 make
 * theirs on the first wave alone: a window at a time where that takes less
 * (a linear rec_tbl and many steps), else in steps without a workgroup
 * barrier, each lane's pos tap in a register (the word a lane makes is its
 * own tap W words later).  Every thread then tempers its own word.  512
 * mexp-11213 streams of 32,768 words, 256 threads: 268 us with W = 2 among
 * them, 93 us all W = 60 (a step at a time: 1546 and 123 us). */
template <bool F32>
__device__ inline uint32_t mtgp_device_draw_bits(mtgp_device_stream &s, uint32_t n) {
    const uint32_t T = blockDim.x, tid = threadIdx.x;
    uint32_t *buf = s.buf;
    const uint32_t *tbl = s.buf + s.cap;
    if (s.h + T > s.cap) {
        // every thread is done with the previous draw's words; cap >= 2N + T,
        // so the last N words never overlap the front
        __syncthreads();
        uint32_t v[4];
        for (uint32_t i0 = 0; i0 < s.N; i0 += 4 * T) {
            for (int j = 0; j < 4; ++j) {
                const uint32_t i = i0 + j * T + tid;
                v[j] = i < s.N ? buf[s.h - s.N + i] : 0u;
            }
            for (int j = 0; j < 4; ++j) {
                const uint32_t i = i0 + j * T + tid;
                if (i < s.N) buf[i] = v[j];
            }
        }
        __syncthreads();
        s.h = s.N;
    }
    const uint32_t h0 = s.h;
    if (s.W < 64u) {
        if (tid < 64u && s.win_e && n > MTGP_DEVICE_WIN_STEPS * s.W) {
            for (uint32_t o = 0; o < n; o += s.win_n)
                mtgp_device_window(s, h0 + o, n - o < s.win_n ? n - o : s.win_n);
        } else if (tid < 64u) {
            if (s.lin) mtgp_device_steps<true>(s, h0, n);
            else mtgp_device_steps<false>(s, h0, n);
        }
    } else {
        const uint32_t smax = s.W < T ? s.W : T;
        for (uint32_t o = 0; o < n; o += smax) {
            const uint32_t S = (n - o) < smax ? (n - o) : smax;
            if (tid >= o && tid < o + S) {
                const uint32_t k = h0 + tid;
                uint32_t X = (buf[k - s.N] & s.mask) ^ buf[k - s.N + 1];
                X ^= X << s.sh1;
                const uint32_t Y = X ^ (buf[k - s.W] >> s.sh2);
                buf[k] = Y ^ tbl[Y & 15u];
            }
            __syncthreads();
        }
    }
    __syncthreads();
    uint32_t result = 0;
    if (tid < n) {
        const uint32_t k = h0 + tid;
        const uint32_t x = buf[k];
        uint32_t H = buf[k - s.W - 1];
        H ^= H >> 16;
        H ^= H >> 8;
        if (F32)
            result = __float_as_uint(__uint_as_float((x >> 9) ^ tbl[32 + (H & 15u)]) - 1.0f);
        else
            result = x ^ tbl[16 + (H & 15u)];
    }
    s.h = h0 + n;
    return result;
}

__device__ inline uint32_t mtgp_device_draw_u32(mtgp_device_stream &s, uint32_t n) {
    return mtgp_device_draw_bits<false>(s, n);
}

__device__ inline float mtgp_device_draw_f32(mtgp_device_stream &s, uint32_t n) {
    return __uint_as_float(mtgp_device_draw_bits<true>(s, n));
}

/* Stores the stream's state (the last N words) to d_state[0..N). */
__device__ inline void mtgp_device_end(mtgp_device_stream &s, uint32_t *d_state) {
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < s.N; i += blockDim.x) d_state[i] = s.buf[s.h - s.N + i];
}

#endif /* MTGP_DEVICE_H */
