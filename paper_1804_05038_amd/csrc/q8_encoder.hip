// q8_encoder.hip -- the encoder recurrence (Eq. 1) of many sentences side by side in one launch: blocks keep their
// recurrent weights in registers for all positions and hand the states to each other through memory.
#include "q8_internal.h"
#include "q8_index.h"
#include <atomic>
#include <mutex>
#include <type_traits>

// Block `member` of a set owns hidden units 32 member .. + 31 of one direction, for the set's sentences ("slots"), in
// groups of up to 16, one group after the other at every time step.  A time step of a group:
//   a wave polls the states that the members of the set published for a slot at the step before (one wave, so that the
//   slot's maximum needs no other wave), quantizes them and leaves the codes in LDS;
//   wave (rt, kp), rt = 2 gate + unit tile, of the first twelve multiplies its 16 weight rows by one half of the k range
//   (at most 512 bytes), the sums cross to the (slot, unit) threads through LDS;
//   the first eight waves apply the gates, store the new states and publish them.
// Arithmetic of quantize_rows_kernel, the panel products and enc_gates_kernel, value for value.
//
// ONE: one group per set (up to 64 sentences of 1024 units).  Every wave has one slot, those without gates the first eight, and
// with XS > 0 the twelve also multiply the rows of X, whose codes and scales the launch in front made, by the block's rows of
// Wx, which lie in LDS (XS k steps of 64 bytes per half): a step's products of X are made while the words of the step before
// travel.  Else (rows of more than 640 bytes) they come from a product launch.  64 sentences of E = 512: 217 us with the
// products given, 182 so (product launches and their 57 MB of results: 41 us).
// Several groups: eight waves take two slots each, eight apply the gates, and the next group's words are requested before this
// one's products; bound by instructions and LDS traffic, so the products of X stay outside (200 sentences: 614 us, 717 with
// them inside).
//
// What orders the accesses to LDS: two barriers per iteration (a group's time step), behind the codes and behind the products.
// Codes are written in front of the first and read between the two, sums written between the two and read behind the second,
// states belong to one thread.  Scales are written in front of the first barrier and read behind the second, where other
// waves are on the next iteration's scales already; so two sets of them take turns (q8_enc_scale).  Rows of X go to LDS at the
// start of an iteration (two turns), are multiplied behind the second barrier of it (sums in two turns) and count in the next
// one, their scales in four turns (q8_enc_x_scale).  A host test walks these accesses.
//
// Exchange with one group.  The members of a set are block numbers that agree modulo 8, which are dealt to one XCD.  Each says
// where it runs; if all are on one XCD, words are stored plainly and loaded past the compute unit's own cache (nt), so both
// ends meet in the XCD's L2: 64 KB per block and step arrive in 0.5 us whenever they are asked for, where agent-scope loads
// (which everybody uses if the members are spread) take 1.1 to 2.4 us, the longer the earlier they ask (16 MB per step
// beyond the L2).  A word is the float with the turn of its buffer, two buffers used twice each, in the bit that no state
// needs (states lie in [-1, 1], whatever X holds: tanh and sigmoid of a NaN are numbers here): whoever polls a word takes none
// of an earlier turn, whatever a cache may still hold, since a location never goes back to an earlier value.  A buffer is free for step t when
// this block has read step t - 1: every member had then read step t - 2.  64 sentences, the same kernel with agent-scope
// loads and stores (q8_encoder_options, one_launch = 2): 263 us; plain stores and nt loads, timed in turn with it: 161.
// With several groups the words' way is hidden, and agent scope is no slower: a word is the float itself, or ENCG_ABSENT (a NaN
// pattern that is never published) while it is not there, three buffers take turns, and a block that has read the words of step
// t - 1 puts its own of step t - 2 back to ENCG_ABSENT, for step t + 1 to be published there, and waits for those stores before
// it publishes step t: whoever polls for step t + 1 has seen step t, and so no word of step t - 2.
//
// Nobody has to be resident for the result to be right.  A wait is bounded; a member that gives up says so in the set's
// flag, at which the others leave as well, and the last member to leave works the whole set off by itself, from the
// first position on, without waiting for anybody.  Words that are not there make no codes: whatever a member stores or
// publishes before it leaves is what the last one stores again.  That is slow (4 ms at 64 sentences), so the blocks of two
// encoders don't compete for the compute units: the launch that clears the words also waits for its turn on the device, and
// the encoder's last block to start passes it on, when all of them are on their units and wait for nobody else.  Four
// streams with a batch of 64 sentences each, us per batch: 2110 without turns (an encoder that ends makes room for part of
// the next two, which wait for each other's room until both give up), 215 with them (a launch per position, before: 358).
//
// The chain of a step bounds it (1024 units, 16 slots, in us behind the second barrier: states published 0.6, words there 1.5,
// codes 1.9, products 2.5, that is the next barrier), with several groups the instructions of the codes and the gates
// (2.6 us per group).  q8_encode_batch, sentences of 10 to 60 words, E = 512, H = 1024, us: 4 / 16 / 32 / 64 / 200 sentences
// 134 / 168 / 192 / 237 / 676 with agent-scope words, four groups' order of waves for all, and the products of X outside;
// 118 / 141 / 159 / 182 / 614 so.  A launch per position: 411 at 64, 880 at 200.
// Not kept: waves of one unit tile and a quarter of the k range that multiply all three gates (a third of the LDS reads,
// more sums to add up: 1 us faster in nothing, 5 slower where a poll comes early); all floats of a step exchanged as
// (float, tag) pairs (twice the bytes); two slots per wave on half of the waves with one group (208 us: a slot's codes are a chain).
#define ENCG_UNITS Q8_ENC_UNITS
#define ENCG_SLOTS Q8_ENC_SLOTS
#define ENCG_THREADS 1024
#define ENCG_PITCH Q8_ENC_PITCH
#define ENCG_TILE Q8_ENC_TILE
#define ENCG_ABSENT 0xffffffffu
#define ENCG_X_LD 640
#define ENCG_SPINS 4096                // polls of a wait at most (some 5 ms; four times as many within an XCD): what follows is slow, not wrong
#define ENCG_AGENT 0x10                 // cache policy of a device-coherent load or store (sc1)
#define ENCG_XCD 2                      // ... of a load that is not served from the compute unit's own cache but from its XCD's (nt)
#define ENCG_TURN_BIT 0x40000000u
#define ENCG_XCC_ID (20 | 3 << 11)      // hardware register XCC_ID, bits 3:0

// The turn on a device (a module's variable, so one per device and process): how many of the last eight blocks (one per XCD;
// blocks of lower index start earlier) of the encoder whose turn it is have started.  Whoever takes an eight from it has the
// next turn; fewer are put back.  The wait ends after ENCG_TURN of the 100 MHz clock (an encoder that failed to launch, or
// whose blocks wait for room behind long kernels): whoever goes on then passes on an eight of its own, so nobody else
// waits for what never comes.  40 ms: an encoder whose blocks wait for room waits for another to end, and 512 sentences of
// 1024 words, the most that one launch takes, are 28 ms.
#define ENCG_TURN 4000000ull
__device__ unsigned enc_group_turn = 8;

// Waits for the turn (block 0), clears [words, words + n) (the next `clear` blocks) and quantizes the L rows of X (E floats, at
// most 1024; the blocks after those, a wave per row), codes at pitch ld.
__global__ __launch_bounds__(256) void enc_group_front_kernel(unsigned *words, int n, int clear, const float *X, int E, int L, int ld, int8_t *xq, float *xs)
{
    if ((int)blockIdx.x > clear) {
        const int row = __builtin_amdgcn_readfirstlane(((int)blockIdx.x - 1 - clear) * 4 + (int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
        if (row >= L) return;
        const __amdgpu_buffer_rsrc_t rx = q8_rsrc(X + (size_t)row * E, (size_t)E * sizeof(float));
        constexpr int C = 4;
        float4 v[C];
        float m = 0.0f;
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rx, (c * 64 + lane) * 16, 0, 0));
#pragma unroll
        for (int c = 0; c < C; ++c) m = fmaxf(m, fmaxf(fmaxf(fabsf(v[c].x), fabsf(v[c].y)), fmaxf(fabsf(v[c].z), fabsf(v[c].w))));
        float scale, inv;
        q8_scale_of(wave_max_f(m), scale, inv);
        if (lane == 0) xs[row] = scale;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int k = (c * 64 + lane) * 4;                         // (zeros past E)
            if (k < ld) *(int *)(xq + (size_t)row * ld + k) = q8_pack4(v[c].x, v[c].y, v[c].z, v[c].w, inv);
        }
        return;
    }
    if (blockIdx.x > 0) {
        const int e = ((int)blockIdx.x - 1) * 256 + (int)threadIdx.x;
        if (e < n) words[e] = ENCG_ABSENT;
        return;
    }
    if (threadIdx.x > 0) return;
    auto take = [] {
        const unsigned had = __hip_atomic_exchange(&enc_group_turn, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (had < 8 && had > 0) __hip_atomic_fetch_add(&enc_group_turn, had, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return had >= 8;
    };
    if (take()) return;
    const unsigned long long begin = wall_clock64();
    while (wall_clock64() - begin < ENCG_TURN) {
        __builtin_amdgcn_s_sleep(16);
        if (__hip_atomic_load(&enc_group_turn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= 8 && take()) return;
    }
}

struct EncGroupArgs {
    const int8_t *Wh[2], *Wht[2];        // [3H x ld], the same tile-packed or NULL
    const float *bh[2], *gx[2];          // [3H] or NULL; XS == 0: [L x 3H]
    const int8_t *Wx[2], *Wxt[2];        // XS > 0: [3H x ldx], the same tile-packed or NULL
    const float *bx[2];                  // [3H] or NULL
    const int8_t *xq;                    // codes [L x ldx] and scales [L] of X
    const float *xs;
    const int *sent_off;                 // [S + 1]
    float *enc_h;                        // [L x 2H]
    unsigned *words;                     // [2 turns, 3 with several groups][2 directions][S][H], the first two ENCG_ABSENT on entry
    unsigned *ctl;                       // [sets][2]: members that left, a wait that gave up; [sets][32]: the XCD of each member; ENCG_ABSENT on entry
    int S, H, ld, members, sets_per_dir, spin_limit, far;               // far: as if the members were not all on one XCD
    float wh_scale[2];
    int ldx;
    float wx_scale[2];
};

// The matrix cores' operands of 16 rows of a gate, N k steps of 64 bytes from step k0 on: units unit0 .. of a matrix of H units,
// pitch bytes per row, tile-packed in Wt if that is there (zeros past H, and past the row).
template <int N>
__device__ __forceinline__ void enc_rows(const int8_t *W, const int8_t *Wt, int pitch, int H, int gate, int unit0, int k0, int lane, v4i (&out)[N])
{
    const int i = lane & 15, gq = lane >> 4;
    const bool tiled = Wt != nullptr && H % 16 == 0;                   // (a tile of 16 rows then belongs to one gate)
    const __amdgpu_buffer_rsrc_t rw = q8_rsrc(tiled ? Wt : W, (size_t)(tiled ? (3 * H + 15) / 16 * 16 : 3 * H) * pitch);
    const unsigned row0 = (unsigned)(gate * H + unit0), step = tiled ? 1024u : 64u;
    const unsigned base = tiled ? ((row0 >> 4) * (unsigned)(pitch >> 6) << 10) + 16u * lane : (row0 + i) * (unsigned)pitch + 16u * gq;
    const bool ok = (tiled ? unit0 : unit0 + i) < H;
#pragma unroll
    for (int s = 0; s < N; ++s) {
        const int k = k0 + s;
        const unsigned off = ok && 64 * k + (tiled ? 0 : 16 * gq) < pitch ? base + step * k : Q8_OOB;
        out[s] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)off, 0, 0));
    }
}

template <int XS, bool ONE>
__global__ __launch_bounds__(ENCG_THREADS) void enc_group_kernel(EncGroupArgs a)
{
    static_assert(XS == 0 || ONE, "rows of X are multiplied for one group at a time");
    extern __shared__ __align__(16) int8_t s_codes[];                  // [16][ENCG_PITCH], sums, states, offsets, lengths; what XS adds
    __shared__ float s_scale[2 * ENCG_SLOTS], s_xs[4 * ENCG_SLOTS];
    __shared__ float s_bias[6][ENCG_UNITS];
    __shared__ int s_flag, s_max, s_far;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, gq = lane >> 4;
    const int H = a.H, S = a.S, ld = a.ld, members = a.members;
    const int round = (int)blockIdx.x >> 3, member = round % members, set = ((int)blockIdx.x & 7) + 8 * (round / members);
    if (blockIdx.x + 8 >= gridDim.x && tid == 0) __hip_atomic_fetch_add(&enc_group_turn, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (set >= 2 * a.sets_per_dir) return;
    // the set's slots, in groups of gs
    const int d = set & 1, c0 = S * (set >> 1) / a.sets_per_dir, ns = S * ((set >> 1) + 1) / a.sets_per_dir - c0;
    const int ng = ONE ? 1 : (ns + ENCG_SLOTS - 1) / ENCG_SLOTS, gs = ONE ? ns : (ns + ng - 1) / ng;
    int *s_e = (int *)(s_codes + ENCG_SLOTS * ENCG_PITCH);
    float *s_h = (float *)(s_e + 12 * ENCG_TILE);                      // [ng][16][32] this block's states
    int *s_off = (int *)(s_h + ng * ENCG_SLOTS * ENCG_UNITS), *s_len = s_off + ng * ENCG_SLOTS;      // [ng][16]
    constexpr int XP = Q8_ENC_X_PITCH(XS);
    int8_t *s_xc = (int8_t *)(s_len + ng * ENCG_SLOTS);                // [2][16][XP]
    int *s_ex = (int *)(s_xc + 2 * ENCG_SLOTS * XP);                   // [2][12 tiles]
    int8_t *s_wx = (int8_t *)(s_ex + 2 * 12 * ENCG_TILE);              // [12 waves][XS][64 lanes] 16 bytes of the rows of Wx
    const int *where = (const int *)(a.ctl + 2 * 2 * a.sets_per_dir + 32 * set);              // the XCD of every member, once it has started
    const int xcd = (int)__builtin_amdgcn_s_getreg(ENCG_XCC_ID);
    if (tid == 0) {
        s_flag = 0;
        s_max = 0;
        __hip_atomic_store((int *)where + member, xcd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    for (int e = tid; e < ng * ENCG_SLOTS; e += ENCG_THREADS) {
        const int in = e & (ENCG_SLOTS - 1), slot = (e >> 4) * gs + in;
        const bool ok = in < gs && slot < ns;                          // (no slot: length 0)
        const int o = ok ? a.sent_off[c0 + slot] : 0, l = ok ? a.sent_off[c0 + slot + 1] - o : 0;
        s_off[e] = o;
        s_len[e] = l;
        atomicMax(&s_max, l);
    }
    for (int e = tid; e < ng * ENCG_SLOTS * ENCG_UNITS; e += ENCG_THREADS) s_h[e] = 0.0f;

    // ---- the parts of a time step ----
    const int rt = wave % 6, kp = wave / 6, gate = rt >> 1, ut = rt & 1;                  // (waves 12 to 15 multiply nothing)
    v4i av[8];
    auto weights = [&](int u0) {
        enc_rows(a.Wh[d], a.Wht[d], ld, wave < 12 ? H : 0, gate, u0 + 16 * ut, kp * 8, lane, av);
        if constexpr (XS > 0) {
            v4i xv[XS];
            enc_rows(a.Wx[d], a.Wxt[d], a.ldx, wave < 12 ? H : 0, gate, u0 + 16 * ut, kp * XS, lane, xv);
            if (wave < 12) {
#pragma unroll
                for (int s = 0; s < XS; ++s) *(v4i *)(s_wx + ((wave * XS + s) * 64 + lane) * 16) = xv[s];
            }
        }
    };
    // of the 32 units from u0 on, by the block's first 32 threads (in front of a barrier); absent ones are the zero that
    // changes no sum
    auto biases = [&](int u0) {
        if (tid < ENCG_UNITS) {
            const int unit = u0 + tid;
#pragma unroll
            for (int gt = 0; gt < 3; ++gt) {
                s_bias[gt][tid] = a.bh[d] && unit < H ? a.bh[d][gt * H + unit] : -0.0f;
                s_bias[3 + gt][tid] = XS > 0 && a.bx[d] && unit < H ? a.bx[d][gt * H + unit] : -0.0f;
            }
        }
    };
    // one wave, iteration it (groups of time steps, counted): the codes and the scales of N slots' states, floats 4 (lane + 64 c) ..
    auto codes = [&](auto &w, int slot, int it) {
        constexpr int N = sizeof(w) / sizeof(w[0]);
        float m[N], scale[N], inv[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            m[q] = 0.0f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m[q]) : "v"(w[q][c].x), "v"(w[q][c].y));
                asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m[q]) : "v"(w[q][c].z), "v"(w[q][c].w));
            }
            m[q] = wave_max_f(m[q]);
        }
#pragma unroll
        for (int q = 0; q < N; ++q) {
            q8_scale_of(m[q], scale[q], inv[q]);
            if (lane == 0) s_scale[q8_enc_scale(it, slot + q)] = scale[q];
        }
#pragma unroll
        for (int q = 0; q < N; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float4 v = __builtin_bit_cast(float4, w[q][c]);
                *(int *)(s_codes + (slot + q) * ENCG_PITCH + 4 * (lane + 64 * c)) = q8_pack4(v.x, v.y, v.z, v.w, inv[q]);
            }
    };
    // (k steps past the rows have zero weights: whatever the codes are there, they add nothing, and no branch makes the wave
    // wait for every operand by itself)
    auto products = [&]() {
        if (wave < 12) {
            v4i acc[2] = {(v4i){0, 0, 0, 0}, (v4i){0, 0, 0, 0}}, bv[8];
            const int8_t *bp = s_codes + i * ENCG_PITCH + kp * 512 + 16 * gq;
#pragma unroll
            for (int s = 0; s < 8; ++s) bv[s] = *(const v4i *)(bp + 64 * s);
#pragma unroll
            for (int s = 0; s < 8; ++s) acc[s & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[s], bv[s], acc[s & 1], 0, 0, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);         // every operand is requested before the first is waited for
            __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
            // lane (i, gq) holds units 4 gq + r, r = 0..3, of slot i
            *(v4i *)(s_e + wave * ENCG_TILE + i * 16 + 4 * gq) = acc[0] + acc[1];
        }
    };
    // the same rows of Wx times the codes of iteration it's rows of X
    auto xproducts = [&](int it) {
        if (XS > 0 && wave < 12) {
            v4i acc[2] = {(v4i){0, 0, 0, 0}, (v4i){0, 0, 0, 0}};
            const int8_t *bp = s_xc + ((it & 1) * ENCG_SLOTS + i) * XP + kp * XS * 64 + 16 * gq, *ap = s_wx + (wave * XS * 64 + lane) * 16;
#pragma unroll
            for (int s = 0; s < XS; ++s)
                acc[s & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(*(const v4i *)(ap + 1024 * s), *(const v4i *)(bp + 64 * s), acc[s & 1], 0, 0, 0);
            *(v4i *)(s_ex + ((it & 1) * 12 + wave) * ENCG_TILE + i * 16 + 4 * gq) = acc[0] + acc[1];
        }
    };
    // a wave's row of X: 16 bytes of codes per lane (lanes past it the last ones again), and the scale
    v4i xr;
    float xsr;
    auto xrequest = [&](int pos) {
        xr = *(const v4i *)(a.xq + (size_t)pos * a.ldx + min(16 * lane, a.ldx - 16));
        xsr = a.xs[pos];
    };
    auto xleave = [&](int slot, int it) {
        if (16 * lane < 128 * XS) *(v4i *)(s_xc + ((it & 1) * ENCG_SLOTS + slot) * XP + 16 * lane) = xr;
        if (lane == 0) s_xs[q8_enc_x_scale(it, slot)] = xsr;
    };
    const int sl = tid >> 5, u = tid & 31;                             // this thread's (slot, unit) pair, below 16 x 32
    float wh_scale = a.wh_scale[d], wx_scale = a.wx_scale[d];
    asm volatile("" : "+v"(wh_scale), "+v"(wx_scale));                 // (kept, not read again at every step)
    // (XS == 0: gx_in the input pre-activations)
    auto gates = [&](const float (&gx_in)[3], float h_prev, int it) {
        int eh[6], ex[6];
        float b[6], gh[3], gx[3];
#pragma unroll
        for (int gt = 0; gt < 3; ++gt) {
            const int at = (gt * 2 + (u >> 4)) * ENCG_TILE + sl * 16 + (u & 15);
            eh[gt] = s_e[at];
            eh[3 + gt] = s_e[at + 6 * ENCG_TILE];
            b[gt] = s_bias[gt][u];
            if (XS > 0) {
                ex[gt] = s_ex[(it & 1) * 12 * ENCG_TILE + at];
                ex[3 + gt] = s_ex[((it & 1) * 12 + 6) * ENCG_TILE + at];
                b[3 + gt] = s_bias[3 + gt][u];
            }
        }
        const float ch = wh_scale * s_scale[q8_enc_scale(it, sl)], cx = XS > 0 ? wx_scale * s_xs[q8_enc_x_scale(it, sl)] : 0.0f;
#pragma unroll
        for (int gt = 0; gt < 3; ++gt) {
            const float y = (float)(eh[gt] + eh[3 + gt]) * ch;
            gh[gt] = y + b[gt];
            if (XS > 0) {
                const float x = (float)(ex[gt] + ex[3 + gt]) * cx;
                gx[gt] = x + b[3 + gt];
            } else {
                gx[gt] = gx_in[gt];
            }
        }
        return gru_gates(gx, gh, h_prev);
    };
    auto input = [&](int pos, int unit, float (&gx)[3]) {
        const float *gp = a.gx[d] + (size_t)pos * 3 * H + unit;
#pragma unroll
        for (int gt = 0; gt < 3; ++gt) gx[gt] = gp[gt * H];
    };
    // row of enc_h (and of gx) of step t of a slot of length l that begins at o, and the row before it
    auto row = [&](int o, int l, int t) { return d == 0 ? o + t : o + l - 1 - t; };
    const int back = d == 0 ? -1 : 1, col0 = d == 0 ? H : 0;

    // ---- all positions ----
    const int unit = member * ENCG_UNITS + u;
    const bool pair = unit < H;                                        // (of the first eight waves: a (slot, unit) pair per thread)
    // words of this direction: byte offset of a buffer; all below 2^31
    const unsigned size = (unsigned)S * (unsigned)H * 8u, dir = d * (size >> 1);
    const __amdgpu_buffer_rsrc_t rx = q8_rsrc(a.words, (size_t)(ONE ? 2 : 3) * size);
    const unsigned mine = (unsigned)((c0 + sl) * H + unit) * 4u;
    // a wait for words that are not there ends: this member leaves, or another has
    auto give_up = [&](int spins, int limit) {
        if (spins < limit &&
            ((spins & 63) != 0 || __hip_atomic_load(a.ctl + 2 * set + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ENCG_ABSENT)) return false;
        if (lane == 0) {
            s_flag = 1;
            __hip_atomic_store(a.ctl + 2 * set + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return true;
    };
    if constexpr (ONE) {
        // ---- one group: a wave per slot, the waves without gates first ----
        biases(member * ENCG_UNITS);
        weights(member * ENCG_UNITS);
        if (wave == 15) {
            // whether every member runs on this XCD
            int far = 1;
            for (int spins = 1;; ++spins) {
                const int x = lane < members ? __hip_atomic_load(where + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : xcd;
                if (!__any(x == (int)ENCG_ABSENT)) {
                    far = a.far || __any(x != xcd);
                    break;
                }
                if (give_up(spins, a.spin_limit)) break;
            }
            if (lane == 0) s_far = far;
        }
        __syncthreads();
        const bool far = s_far != 0;
        const int slot = wave ^ 8, max_l = s_max;
        const int wl = __builtin_amdgcn_readfirstlane(s_len[slot]), wo = __builtin_amdgcn_readfirstlane(s_off[slot]);
        const int tl = s_len[min(sl, ENCG_SLOTS - 1)], to = s_off[min(sl, ENCG_SLOTS - 1)];
        auto buffer = [&](int t) { return (unsigned)(t & 1) * size + dir; };
        auto turn = [&](int t) { return (unsigned)(t & 2) << 29; };    // the bit of a turn's words
        auto xpos = [&](int t) { return t < wl ? row(wo, wl, t) : 0; };
        // rows of X: requested behind a step's words, whose wait theirs would prolong, left in LDS at the start of the next
        // step and multiplied at the end of that, for the one after
        if (XS > 0) {
            xrequest(xpos(0));
            xleave(slot, 0);
            xrequest(xpos(1));
            __syncthreads();
            xproducts(0);
        }
        float h_prev = 0.0f, gx[3] = {0.f, 0.f, 0.f};
        auto ahead = [&](int t) { input(pair && t < tl ? row(to, tl, t) : 0, pair ? unit : 0, gx); };     // the pre-activations of a step to come
        if (XS == 0) ahead(0);
        for (int t = 0; t < max_l; ++t) {
            if (XS > 0) xleave(slot, t + 1);
            if (t < wl) {                                              // wave-uniform
                v4u w[1][4];
                bool there = true;
                auto poll = [&](auto policy) {                         // (past H: the last ones again, for weights of zero)
                    if (decltype(policy)::value == ENCG_AGENT) __builtin_amdgcn_s_sleep(8);    // (too early a poll slows what it waits for)
                    const int from = (int)(buffer(t - 1) + (unsigned)((c0 + slot) * H) * 4u);
                    unsigned first = 16u * lane, m = 0;
                    asm volatile("" : "+v"(first) :: "memory");        // (every request is made)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        w[0][c] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)min(first + 1024u * c, 4u * H - 16u), from, decltype(policy)::value));
                    // what is there is the state itself once its turn's bit is off
                    const unsigned bit = turn(t - 1);
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        w[0][c] ^= bit;
                        m |= w[0][c].x | w[0][c].y | w[0][c].z | w[0][c].w;
                    }
                    return !__any((m & ENCG_TURN_BIT) != 0);
                };
                if (t > 0) {
                    if (far) {
                        for (int spins = 1; !(there = poll(std::integral_constant<int, ENCG_AGENT>())) && !give_up(spins, a.spin_limit); ++spins) {}
                    } else {
                        for (int spins = 1; !(there = poll(std::integral_constant<int, ENCG_XCD>())) && !give_up(spins, a.spin_limit < ENCG_SPINS ? a.spin_limit : 4 * ENCG_SPINS); ++spins) {}
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) w[0][c] = (v4u){0u, 0u, 0u, 0u};
                }
                if (XS > 0) xrequest(xpos(t + 2));
                if (there) codes(w, slot, t);
            }
            __syncthreads();
            const int flag = s_flag;
            const float gx_now[3] = {gx[0], gx[1], gx[2]};
            if (XS == 0) ahead(t + 1);
            products();
            __syncthreads();
            if (flag) break;
            if (wave < 8) {
                __builtin_amdgcn_s_setprio(2);                         // everybody waits for them
                const float hn = gates(gx_now, h_prev, t);
                if (pair && t < tl) {
                    const unsigned word = __float_as_uint(hn) ^ turn(t);
                    const int at = (int)(mine + buffer(t));
                    if (t + 1 < tl) {
                        if (far) __builtin_amdgcn_raw_buffer_store_b32(word, rx, at, 0, ENCG_AGENT);
                        else __builtin_amdgcn_raw_buffer_store_b32(word, rx, at, 0, 0);
                    }
                    a.enc_h[(size_t)row(to, tl, t) * 2 * H + col0 + unit] = hn;
                    h_prev = hn;
                }
                __builtin_amdgcn_s_setprio(0);
            }
            xproducts(t + 1);
        }
    } else {
        // ---- several groups, one after the other at every step: the gates on the first eight waves, the codes, of two slots
        // each, on the others ----
        weights(member * ENCG_UNITS);
        biases(member * ENCG_UNITS);
        __syncthreads();
        const int max_l = s_max;
        const unsigned group = (unsigned)(gs * H) * 4u;
        auto buffer = [&](int t) { return (unsigned)(t % 3) * size + dir; };
        bool gave_up = false;
        int it = 0;
        if (wave < 8) {
            float gx[3] = {0.f, 0.f, 0.f};
            auto ahead = [&](int t, int g) {                           // the pre-activations of an iteration to come
                const int e = g * ENCG_SLOTS + sl, l = s_len[e];
                input(pair && t < l ? row(s_off[e], l, t) : 0, pair ? unit : 0, gx);
            };
            ahead(0, 0);
            for (int t = 0; t < max_l && !gave_up; ++t) {
                for (int g = 0; g < ng; ++g, ++it) {
                    const int e = g * ENCG_SLOTS + sl, l = s_len[e], pos = row(s_off[e], l, t);
                    const float h_prev = s_h[g * ENCG_SLOTS * ENCG_UNITS + tid];
                    const int at = (int)(mine + g * group);
                    __syncthreads();
                    const int flag = s_flag;
                    if (pair && t + 2 < l && !flag) __builtin_amdgcn_raw_buffer_store_b32(ENCG_ABSENT, rx, at, (int)buffer(t + 1), ENCG_AGENT);
                    products();
                    __syncthreads();
                    if (flag) { gave_up = true; break; }
                    __builtin_amdgcn_s_setprio(2);
                    const float hn = gates(gx, h_prev, it);
                    if (pair && t < l) {
                        unsigned word = __float_as_uint(hn);
                        word = word == ENCG_ABSENT ? 0x7fffffffu : word;
                        q8_stores_performed();
                        if (t + 1 < l) __builtin_amdgcn_raw_buffer_store_b32(word, rx, at, (int)buffer(t), ENCG_AGENT);
                        a.enc_h[(size_t)pos * 2 * H + col0 + unit] = hn;
                        s_h[g * ENCG_SLOTS * ENCG_UNITS + tid] = hn;
                    }
                    __builtin_amdgcn_s_setprio(0);
                    ahead(g + 1 == ng ? t + 1 : t, g + 1 == ng ? 0 : g + 1);
                }
            }
        } else {
            const int pair0 = 2 * (wave - 8);
            auto len = [&](int g, int q) { return __builtin_amdgcn_readfirstlane(s_len[g * ENCG_SLOTS + pair0 + q]); };
            // floats 4 (lane + 64 c) .. of the first (past H: zero, which is there)
            unsigned at[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) at[c] = 4 * (lane + 64 * c) < H ? (unsigned)((c0 + pair0) * H + 4 * (lane + 64 * c)) * 4u : Q8_OOB;
            v4u w[2][4];
            // step t's of group g: the words of step t - 1 (none at step 0, and of a sentence that is over: zeros)
            auto request = [&](int t, int g) {
                asm volatile("" ::: "memory");                         // (every request is made)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const unsigned from = t > 0 && t < len(g, q) ? buffer(t - 1) + g * group + (unsigned)(q * H) * 4u : Q8_OOB;
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        w[q][c] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(at[c] == Q8_OOB || from == Q8_OOB ? Q8_OOB : at[c] + from), 0, ENCG_AGENT));
                }
            };
            request(0, 0);
            for (int t = 0; t < max_l && !gave_up; ++t) {
                for (int g = 0; g < ng; ++g, ++it) {
                    bool there = true;
                    for (int spins = 1;; ++spins) {
                        unsigned m = 0;                                // (an absent word is the largest there is)
#pragma unroll
                        for (int q = 0; q < 2; ++q)
#pragma unroll
                            for (int c = 0; c < 4; ++c) m = max(max(m, max(w[q][c].x, w[q][c].y)), max(w[q][c].z, w[q][c].w));
                        if (!__any(m == ENCG_ABSENT)) break;
                        if (give_up(spins, a.spin_limit)) {
                            there = false;
                            break;
                        }
                        request(t, g);
                    }
                    if (there) codes(w, pair0, it);
                    __syncthreads();
                    const int flag = s_flag;
                    request(g + 1 == ng ? t + 1 : t, g + 1 == ng ? 0 : g + 1);    // the next group's words, under this one's products and gates
                    products();
                    __syncthreads();
                    if (flag) { gave_up = true; break; }
                }
            }
        }
    }

    // ---- the last member to leave a set in which a wait gave up ----
    q8_stores_performed();
    __syncthreads();
    if (tid == 0) {
        const unsigned before = __hip_atomic_fetch_add(a.ctl + 2 * set, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_flag = before + 2u == (unsigned)members && __hip_atomic_load(a.ctl + 2 * set + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != ENCG_ABSENT;
    }
    __syncthreads();
    if (!s_flag) return;
    for (int g = 0; g < ng; ++g)
        for (int t = 0; t < s_max; ++t) {
            const int e0 = g * ENCG_SLOTS, lw = s_len[e0 + wave], pos0 = t < lw ? row(s_off[e0 + wave], lw, t) : 0;
            v4u v[1][4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int k = 4 * (lane + 64 * c);
                v[0][c] = t > 0 && t < lw && k < H ? *(const v4u *)(a.enc_h + (size_t)(pos0 + back) * 2 * H + col0 + k) : (v4u){0u, 0u, 0u, 0u};
            }
            codes(v, wave, 0);
            if (XS > 0) {
                xrequest(pos0);
                xleave(wave, 0);
            }
            for (int m = 0; m < members; ++m) {
                const int unit = m * ENCG_UNITS + u, at = min(e0 + sl, ng * ENCG_SLOTS - 1), l = s_len[at], pos = row(s_off[at], l, t);
                weights(m * ENCG_UNITS);
                __syncthreads();                                       // (behind the gates of the member before)
                biases(m * ENCG_UNITS);
                products();
                xproducts(0);
                __syncthreads();
                if (sl < ENCG_SLOTS && unit < H && t < l) {
                    float gx[3] = {0.f, 0.f, 0.f};
                    if (XS == 0) input(pos, unit, gx);
                    a.enc_h[(size_t)pos * 2 * H + col0 + unit] = gates(gx, t > 0 ? a.enc_h[(size_t)(pos + back) * 2 * H + col0 + unit] : 0.0f, 0);
                }
            }
            __syncthreads();
        }
}

// ================================================= one sentence, all positions ==
// Eq. 1 of one sentence, both directions, in one launch whose blocks wait for each other.  A direction's blocks are those
// block numbers that agree with it modulo 8 (one XCD); a block of twelve waves owns 32 hidden units and keeps their rows of
// Wh and Wx in registers, wave (rt, kp) as in enc_group_kernel.  A step: four waves (one per SIMD) poll all words of the step
// before, each takes the maximum by itself and leaves a quarter of the codes in LDS; twelve waves multiply (of the matrix
// cores' sixteen columns one is used: that takes no sums across lanes); the fifth wave applies the gates, r in its lower
// half and z in its upper, and publishes.  While the words travel, the next position's products of X are made, from
// rows that lie in LDS, `chunk` at a time.  Words, turns and what the members do when they are spread over several XCDs: as
// in enc_group_kernel with one group.  Arithmetic of quantize_rows_kernel, the products and encoder_persistent_kernel, value for value.
// Nobody has to be resident for the result to be right: a wait is bounded, the first block of a direction whose wait gives up
// works the direction off by itself (enc_one_alone), and the others leave when they next look at its word.  What they stored
// before is what it stores, and it reads no states but its own, so it need not be the last.
// The chain of a step bounds it: 1.50 us per position, E = 512, H = 1024 (encoder_persistent_kernel, 256 blocks all over the
// device: 1.83, and two launches more in front).  q8_encode of 50 words, us: 99 -> 84, with states handed over device-coherently 124; on 1 / 2 / 3 / 4
// streams at once, per sentence, 100 / 128 / 120 / 117 -> 84 / 44 / 44 / 48, E = 64 100 / 126 / 118 / 115 -> 83 / 43 / 49 / 53 (more than two wait for their turns to start).
// Not kept: dot products and gates on every wave, two units of sixteen waves or four of eight (129 and 101 us: sums across
// lanes and sixteen, or eight, waves' gates); a row of X from memory at every step (135: its way is longer than the words').
// LDS between the two barriers of a step: codes, sums and scales as in enc_group_kernel (states are words' own); sums of X
// take turns; rows of X are replaced between two barriers of their own.
struct EncOneArgs {
    const int8_t *Wh[2], *Wht[2], *Wx[2], *Wxt[2];     // [3H x ld], [3H x ldx], and the same tile-packed or NULL
    const float *bh[2], *bx[2];          // [3H] or NULL
    const int8_t *xq;                    // codes [l x ldx] and scales [l] of X
    const float *xs;
    float *enc_h;                        // [l x 2H]
    unsigned *words;                     // [2 turns][2 directions][H], ENCG_ABSENT on entry
    unsigned *ctl;                       // [2][4]: a wait gave up, a block works the direction off; [2][32]: the XCD of each member; ENCG_ABSENT on entry
    unsigned *err;                       // set where the caller's own bound ended a wait
    int l, H, ld, ldx, members, first, spin_limit, chunk, far;
    float wh_scale[2], wx_scale[2];
};
#define ENC1_WAVES 12

// What a block of direction dir does that leaves early (flag 2: the caller's own bound ended its wait): the first one works the
// direction off, all positions and units, a wave per unit as in encoder_persistent_kernel.  q, xq: 1024 bytes of LDS each.
// A position of 1024 units takes it 310 us (64: 13).  (Kept out of the loop of enc_one_kernel, down to the claim, and told to be unlikely: with the
// claim made in the waits, or the loop left through an ordinary branch, a position took 1.55 to 1.70 us in place of 1.50.)
static __device__ __forceinline__ void enc_one_alone(const EncOneArgs *p, int dir, int flag, int8_t *q, int8_t *xq)
{
    const EncOneArgs &a = *p;
    if (threadIdx.x == 0) {
        *(unsigned *)q = __hip_atomic_exchange(a.ctl + 4 * dir + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (flag == 2) __hip_atomic_store(a.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const unsigned before = *(const unsigned *)q;
    __syncthreads();
    if (before != ENCG_ABSENT) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), d = __builtin_amdgcn_readfirstlane(dir);
    const int H = __builtin_amdgcn_readfirstlane(a.H), L = __builtin_amdgcn_readfirstlane(a.l), ld = a.ld, ldx = a.ldx, col0 = d == 0 ? H : 0;
    const v4i none = {0, 0, 0, 0};
    for (int t = 0; t < L; ++t) {
        const int pos = d == 0 ? t : L - 1 - t;
        float *to = a.enc_h + (size_t)pos * 2 * H + col0;
        const float *from = to + (d == 0 ? -2 * H : 2 * H);
        float4 v[4];
        float m = 0.0f, scale, inv;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int k = 4 * (lane + 64 * c);
            v[c] = t > 0 && k < H ? *(const float4 *)(from + k) : make_float4(0.f, 0.f, 0.f, 0.f);
            m = fmaxf(m, fmaxf(fmaxf(fabsf(v[c].x), fabsf(v[c].y)), fmaxf(fabsf(v[c].z), fabsf(v[c].w))));
        }
        q8_scale_of(wave_max_f(m), scale, inv);
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (wave == c) *(int *)(q + 4 * (lane + 64 * c)) = q8_pack4(v[c].x, v[c].y, v[c].z, v[c].w, inv);
        if (wave == 4 && 16 * lane < ldx) *(v4i *)(xq + 16 * lane) = *(const v4i *)(a.xq + (size_t)pos * ldx + 16 * lane);
        const float ch = a.wh_scale[d] * scale, cx = a.wx_scale[d] * a.xs[pos];
        __syncthreads();
        for (int u = wave; u < H; u += ENC1_WAVES) {
            float gx[3], gh[3];
#pragma unroll
            for (int g = 0; g < 3; ++g) {
                const int row = g * H + u;
                const v4i wh = 16 * lane < ld ? *(const v4i *)(a.Wh[d] + (size_t)row * ld + 16 * lane) : none;
                const v4i wx = 16 * lane < ldx ? *(const v4i *)(a.Wx[d] + (size_t)row * ldx + 16 * lane) : none;
                const float y = (float)group_sum_i(dot16(wh, *(const v4i *)(q + 16 * lane), 0), 64) * ch;
                const float x = (float)group_sum_i(dot16(wx, 16 * lane < ldx ? *(const v4i *)(xq + 16 * lane) : none, 0), 64) * cx;
                gh[g] = a.bh[d] ? y + a.bh[d][row] : y;
                gx[g] = a.bx[d] ? x + a.bx[d][row] : x;
            }
            const float hn = gru_gates(gx, gh, t > 0 ? from[u] : 0.0f);
            if (lane == 0) to[u] = hn;
        }
        __syncthreads();
    }
}

template <int XS>
__global__ __launch_bounds__(64 * ENC1_WAVES) void enc_one_kernel(EncOneArgs a)
{
    extern __shared__ __align__(16) int8_t s_x[];                      // [chunk][128 XS] codes of rows of X
    __shared__ __align__(16) int8_t s_q[1024];
    __shared__ __align__(16) int s_e[ENC1_WAVES * 16], s_ex[2][ENC1_WAVES * 16];
    __shared__ float s_scale[2];
    __shared__ int s_flag, s_far;
    constexpr int XP = 128 * XS;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), gq = lane >> 4;
    if (blockIdx.x + 8 >= gridDim.x && tid == 0) __hip_atomic_fetch_add(&enc_group_turn, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int d = ((int)blockIdx.x - a.first) & 7, member = (int)blockIdx.x >> 3, H = a.H;
    if (d > 1) return;
    unsigned *gave_up = a.ctl + 4 * d, *where = a.ctl + 8 + 32 * d;
    const int xcd = (int)__builtin_amdgcn_s_getreg(ENCG_XCC_ID);
    if (tid == 0) {
        s_flag = 0;
        __hip_atomic_store(where + member, (unsigned)xcd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const int rt = wave % 6, kp = wave / 6, unit0 = member * ENCG_UNITS;
    v4i wh[8], wx[XS];
    enc_rows(a.Wh[d], a.Wht[d], a.ld, H, rt >> 1, unit0 + 16 * (rt & 1), kp * 8, lane, wh);
    enc_rows(a.Wx[d], a.Wxt[d], a.ldx, H, rt >> 1, unit0 + 16 * (rt & 1), kp * XS, lane, wx);
    // the gates' wave: unit, and biases of the lane's gate (r or z) and of n
    const int unit = unit0 + (lane & 31);
    const bool is = unit < H;
    float bh[2], bx[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int r = (k == 0 ? lane >> 5 : 2) * H + unit;
        bh[k] = a.bh[d] && is ? a.bh[d][r] : -0.0f;                    // (absent ones are the zero that changes no sum)
        bx[k] = a.bx[d] && is ? a.bx[d][r] : -0.0f;
    }
    auto give_up = [&](int spins, int limit) {
        if (spins < limit && ((spins & 63) != 0 || __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ENCG_ABSENT)) return false;
        if (lane == 0) {
            s_flag = spins < a.spin_limit ? 1 : 2;
            __hip_atomic_store(gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return true;
    };
    __syncthreads();
    if (wave == ENC1_WAVES - 1) {
        int far = 1;
        for (int spins = 1;; ++spins) {
            const int x = lane < a.members ? (int)__hip_atomic_load(where + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : xcd;
            if (!__any(x == (int)ENCG_ABSENT)) {
                far = a.far || __any(x != xcd);
                break;
            }
            if (give_up(spins, min(a.spin_limit, ENCG_SPINS))) break;
        }
        if (lane == 0) s_far = far;
    }
    auto position = [&](int t) { return d == 0 ? t : a.l - 1 - t; };
    auto rows_of_x = [&](int t0) {                                     // those of steps t0 .. (in front of a barrier)
        const int n = min(a.chunk, a.l - t0);
        for (int r = wave; r < n; r += ENC1_WAVES)
            if (16 * lane < XP) *(v4i *)(s_x + r * XP + 16 * lane) = *(const v4i *)(a.xq + (size_t)position(t0 + r) * a.ldx + min(16 * lane, a.ldx - 16));
    };
    auto xproducts = [&](int t, int r) {                               // (lanes of all columns read the same operand)
        v4i acc[2] = {(v4i){0, 0, 0, 0}, (v4i){0, 0, 0, 0}};
        const int8_t *bp = s_x + r * XP + kp * XS * 64 + 16 * gq;
#pragma unroll
        for (int s = 0; s < XS; ++s) acc[s & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wx[s], *(const v4i *)(bp + 64 * s), acc[s & 1], 0, 0, 0);
        if ((lane & 15) == 0) *(v4i *)(s_ex[t & 1] + wave * 16 + 4 * gq) = acc[0] + acc[1];
    };
    rows_of_x(0);
    __syncthreads();
    xproducts(0, 0);
    const bool far = s_far != 0;
    const __amdgpu_buffer_rsrc_t rx = q8_rsrc(a.words, (size_t)16 * H);
    auto buffer = [&](int t) { return (unsigned)((t & 1) * 2 + d) * (unsigned)H * 4u; };
    auto turn = [&](int t) { return (unsigned)(t & 2) << 29; };
    const int limit = far || a.spin_limit < ENCG_SPINS ? a.spin_limit : 4 * ENCG_SPINS;
    float wh_scale = a.wh_scale[d], wx_scale = a.wx_scale[d], h_prev = 0.0f, xs_now = a.xs[position(0)];
    asm volatile("" : "+v"(wh_scale), "+v"(wx_scale));                 // (kept, not read again at every step)
    for (int t = 0, xrow = 0; t < a.l; ++t) {
        if (wave < 4) {
            v4u w[4];                                                  // floats 4 (lane + 64 ((wave + c) % 4)) ..
            bool there = true;
            auto poll = [&](auto policy) {
                if (decltype(policy)::value == ENCG_AGENT) __builtin_amdgcn_s_sleep(8);
                unsigned first = 16u * lane, m = 0;
                asm volatile("" : "+v"(first) :: "memory");            // (every request is made)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    w[c] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)min(first + 1024u * ((wave + c) & 3), 4u * H - 16u), (int)buffer(t - 1), decltype(policy)::value));
                const unsigned bit = turn(t - 1);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    w[c] ^= bit;
                    m |= w[c].x | w[c].y | w[c].z | w[c].w;
                }
                return !__any((m & ENCG_TURN_BIT) != 0);
            };
            if (t > 0) {
                if (far) {
                    for (int spins = 1; !(there = poll(std::integral_constant<int, ENCG_AGENT>())) && !give_up(spins, limit); ++spins) {}
                } else {
                    for (int spins = 1; !(there = poll(std::integral_constant<int, ENCG_XCD>())) && !give_up(spins, limit); ++spins) {}
                }
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) w[c] = (v4u){0u, 0u, 0u, 0u};
            }
            if (there) {
                float m = 0.0f, scale, inv;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(w[c].x), "v"(w[c].y));
                    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(w[c].z), "v"(w[c].w));
                }
                q8_scale_of(wave_max_f(m), scale, inv);
                const float4 v = __builtin_bit_cast(float4, w[0]);
                *(int *)(s_q + 4 * (lane + 64 * wave)) = q8_pack4(v.x, v.y, v.z, v.w, inv);
                if (tid == 0) s_scale[t & 1] = scale;
            }
        }
        __syncthreads();
        const int flag = s_flag;
        {
            v4i acc[2] = {(v4i){0, 0, 0, 0}, (v4i){0, 0, 0, 0}}, bv[8];
            const int8_t *bp = s_q + kp * 512 + 16 * gq;
#pragma unroll
            for (int s = 0; s < 8; ++s) bv[s] = *(const v4i *)(bp + 64 * s);
#pragma unroll
            for (int s = 0; s < 8; ++s) acc[s & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wh[s], bv[s], acc[s & 1], 0, 0, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);         // every operand is requested before the first is waited for
            __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
            if ((lane & 15) == 0) *(v4i *)(s_e + wave * 16 + 4 * gq) = acc[0] + acc[1];
        }
        __syncthreads();
        if (__builtin_expect(flag, 0)) break;
        if (wave == 4) {
            __builtin_amdgcn_s_setprio(2);
            const int u = lane & 31, at[2] = {32 * (lane >> 5) + u, 64 + u};       // sums of the lane's gate and of n (the other half of k 96 further on)
            float gh[2], gx[2];
            int eh[2], ex[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                eh[k] = s_e[at[k]] + s_e[at[k] + 96];
                ex[k] = s_ex[t & 1][at[k]] + s_ex[t & 1][at[k] + 96];
            }
            const float ch = wh_scale * s_scale[t & 1], cx = wx_scale * xs_now;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const float y = (float)eh[k] * ch, x = (float)ex[k] * cx;
                gh[k] = y + bh[k];
                gx[k] = x + bx[k];
            }
            // gru_gates, operation by operation; r and z side by side
            const float sg = sigmoid_rn(gx[0] + gh[0]);
            const auto rz = __builtin_amdgcn_permlane32_swap(__float_as_uint(sg), __float_as_uint(sg), false, false);  // [0]: r, [1]: z
            const float r = __uint_as_float(rz[0]), z = __uint_as_float(rz[1]);
            const float rn = r * gh[1], pn = gx[1] + rn, nn = tanh_rn(pn), omz = 1.0f - z, t1 = omz * nn, t2 = z * h_prev, hn = t1 + t2;
            if (lane < 32 && is) {
                if (t + 1 < a.l) {
                    const unsigned word = __float_as_uint(hn) ^ turn(t);
                    if (far) __builtin_amdgcn_raw_buffer_store_b32(word, rx, unit * 4, (int)buffer(t), ENCG_AGENT);
                    else __builtin_amdgcn_raw_buffer_store_b32(word, rx, unit * 4, (int)buffer(t), 0);
                }
                a.enc_h[(size_t)position(t) * 2 * H + (d == 0 ? H : 0) + unit] = hn;
            }
            __builtin_amdgcn_s_setprio(0);
            h_prev = hn;
            xs_now = a.xs[position(min(t + 1, a.l - 1))];
        }
        if (++xrow == a.chunk) {
            xrow = 0;
            __syncthreads();                                           // (the last one's row has been multiplied)
            if (t + 1 < a.l) rows_of_x(t + 1);
            __syncthreads();
        }
        xproducts(t + 1, xrow);
    }
    if (__builtin_expect(s_flag, 0)) enc_one_alone((const EncOneArgs *)__builtin_amdgcn_kernarg_segment_ptr(), d, s_flag, s_q, s_x);
}

// =================================================================== host launchers ==

// An encoder's two launches side by side on their queue: a stream that shares it cannot wait for the turn between them.
static std::mutex enc_pair;

// 4-byte words of scratch (0: not for this shape): the members' words and the sets' counters and flags.
size_t q8i_enc_group_words(const q8_gru_weights *fwd, const q8_gru_weights *bwd, int S, int max_l)
{
    const int H = fwd->Wh.cols;
    int members, sets, groups, slots;
    if (H % 4 || H > 1024 || fwd->Wh.ld > 1024 || bwd->Wh.ld != fwd->Wh.ld || !q8_enc_one_launch(H, S, max_l)) return 0;
    q8_enc_plan(H, S, &members, &sets, &groups, &slots);
    return (size_t)(groups == 1 ? 4 : 6) * S * H + (4 + 2 * 32) * sets;
}

// Whether the kernel multiplies the rows of X itself (its registers hold the rows of Wx of at most ENCG_X_LD bytes).
bool q8i_enc_group_takes_x(const q8_gru_weights *fwd, int S)
{
    int members, sets, groups, slots;
    q8_enc_plan(fwd->Wh.cols, S, &members, &sets, &groups, &slots);
    return groups == 1 && fwd->Wx.ld <= ENCG_X_LD;
}

template <int XS, bool ONE> static q8_status enc_group_launch(q8_ctx *ctx, const EncGroupArgs &a, int blocks, size_t lds)
{
    static Q8OncePerDevice asked;
    const void *kernel = (const void *)enc_group_kernel<XS, ONE>;
    const q8_status st = q8i_lds(ctx, asked, kernel, Q8_ENC_X_LDS(XS) + Q8_ENC_LDS_MOST, "encoder recurrences");
    if (st) return st;
    Q8_LAUNCH(ctx, Q8_KERNEL_GRU, (enc_group_kernel<XS, ONE>), dim3(blocks), dim3(ENCG_THREADS), lds + Q8_ENC_X_LDS(XS), a);
    return q8i_launch_check(ctx, "encoder recurrences");
}

// in->X: the kernel multiplies the L rows of X, whose codes and scales go to xq [L x ldx] and xs; NULL: gxf, gxb have the products.
q8_status q8i_enc_group(q8_ctx *ctx, const q8_gru_weights *fwd, const q8_gru_weights *bwd, const int *sent_off, int S, float *enc_h,
                        const q8i_enc_input *in, unsigned *words)
{
    const int H = fwd->Wh.cols, L = in->X ? in->L : 0;
    int members, spd, ng, gs;
    const size_t lds = q8_enc_plan(H, S, &members, &spd, &ng, &gs);
    const int clear = (4 + 2 * 32) * spd + 4 * S * H, cb = (clear + 255) / 256;
    EncGroupArgs a = {{fwd->Wh.data, bwd->Wh.data}, {fwd->Wh.tiles, bwd->Wh.tiles}, {fwd->bh, bwd->bh}, {in->gxf, in->gxb},
                      {fwd->Wx.data, bwd->Wx.data}, {fwd->Wx.ld % 64 == 0 ? fwd->Wx.tiles : nullptr, bwd->Wx.ld % 64 == 0 ? bwd->Wx.tiles : nullptr},
                      {fwd->bx, bwd->bx}, in->xq, in->xs, sent_off, enc_h,
                      words + (4 + 2 * 32) * spd, words, S, H, fwd->Wh.ld, members, spd, ctx->enc_spin_limit < ENCG_SPINS ? ctx->enc_spin_limit : ENCG_SPINS, ctx->enc_one_launch == 2,
                      {fwd->Wh.scale, bwd->Wh.scale}, fwd->Wx.ld, {fwd->Wx.scale, bwd->Wx.scale}};
    const int blocks = 8 * members * ((2 * spd + 7) / 8);
    std::lock_guard<std::mutex> hold(enc_pair);
    hipLaunchKernelGGL(enc_group_front_kernel, dim3(1 + cb + (L + 3) / 4), dim3(256), 0, ctx->stream, words, clear, cb, in->X, fwd->Wx.cols, L, fwd->Wx.ld,
                       in->xq, in->xs);
    const q8_status st = q8i_launch_check(ctx, "clear");
    if (st) return st;
    if (!in->X) return ng == 1 ? enc_group_launch<0, true>(ctx, a, blocks, lds) : enc_group_launch<0, false>(ctx, a, blocks, lds);
    return fwd->Wx.ld <= 512 ? enc_group_launch<4, true>(ctx, a, blocks, lds) : enc_group_launch<5, true>(ctx, a, blocks, lds);
}

// Eq. 1 of one sentence in one launch.  Q8_OK with *launched = 0 where the shape is not covered, the device cannot hold all blocks
// at once or the stream is being captured (what it takes then runs elsewhere).  words: q8i_enc_one_words of scratch; xq [l x ldx], xs [l]: room
// for the codes and scales of X; err: set to 1 by the kernel if the context's own bound ended a wait (the states are right all the same).
#define ENC1_CTL (8 + 2 * 32)
size_t q8i_enc_one_words(int H) { return (size_t)4 * H + ENC1_CTL; }

q8_status q8i_enc_one(q8_ctx *ctx, const q8_gru_weights *fwd, const q8_gru_weights *bwd, const float *X, int l, float *enc_h, unsigned *words,
                      int8_t *xq, float *xs, unsigned *err, int *launched)
{
    *launched = 0;
    const int H = fwd->Wh.cols, ldx = fwd->Wx.ld, members = (H + ENCG_UNITS - 1) / ENCG_UNITS, blocks = 8 * members;
    if (H > 1024 || H % 4 || fwd->Wh.ld > 1024 || bwd->Wh.ld != fwd->Wh.ld || ldx > 1024 || bwd->Wx.ld != ldx) return Q8_OK;
    const bool packed = H % 16 == 0 && ldx % 64 == 0 && fwd->Wx.tiles && bwd->Wx.tiles && fwd->Wh.tiles && bwd->Wh.tiles;
    if (!q8_enc_one_better(H, ldx, packed, l)) return Q8_OK;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(ctx->stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) return Q8_OK;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < blocks) {
        (void)hipGetLastError();
        return Q8_OK;
    }
    // sentences on other streams on other XCDs, two at a time
    static std::atomic<unsigned> next{0};
    const int first = 2 * (int)(next.fetch_add(1, std::memory_order_relaxed) & 3), clear = 4 * H + ENC1_CTL, cb = (clear + 255) / 256;
    const int xs4 = ldx <= 512 ? 4 : ldx <= 640 ? 5 : 8, chunk = l < 49152 / (128 * xs4) ? l : 49152 / (128 * xs4);
    EncOneArgs a = {{fwd->Wh.data, bwd->Wh.data}, {fwd->Wh.tiles, bwd->Wh.tiles}, {fwd->Wx.data, bwd->Wx.data},
                    {ldx % 64 == 0 ? fwd->Wx.tiles : nullptr, ldx % 64 == 0 ? bwd->Wx.tiles : nullptr}, {fwd->bh, bwd->bh}, {fwd->bx, bwd->bx}, xq, xs, enc_h,
                    words + ENC1_CTL, words, err, l, H, fwd->Wh.ld, ldx, members, first, ctx->enc_spin_limit, chunk, ctx->enc_one_launch == 2,
                    {fwd->Wh.scale, bwd->Wh.scale}, {fwd->Wx.scale, bwd->Wx.scale}};
    std::lock_guard<std::mutex> hold(enc_pair);
    hipLaunchKernelGGL(enc_group_front_kernel, dim3(1 + cb + (l + 3) / 4), dim3(256), 0, ctx->stream, words, clear, cb, X, fwd->Wx.cols, l, ldx, xq, xs);
    q8_status st = q8i_launch_check(ctx, "clear");
    if (st) return st;
    const dim3 grid(blocks), block(64 * ENC1_WAVES);
    const size_t lds = (size_t)chunk * 128 * xs4;
    if (xs4 == 4) Q8_LAUNCH(ctx, Q8_KERNEL_GRU, enc_one_kernel<4>, grid, block, lds, a);
    else if (xs4 == 5) Q8_LAUNCH(ctx, Q8_KERNEL_GRU, enc_one_kernel<5>, grid, block, lds, a);
    else Q8_LAUNCH(ctx, Q8_KERNEL_GRU, enc_one_kernel<8>, grid, block, lds, a);
    st = q8i_launch_check(ctx, "encoder recurrence");
    if (!st) *launched = 1;
    return st;
}
