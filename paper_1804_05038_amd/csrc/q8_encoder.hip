// q8_encoder.hip -- the encoder recurrence (Eq. 1) of many sentences side by side in one launch: blocks keep their
// recurrent weights in registers for all positions and hand the states to each other through memory.
#include "q8_internal.h"
#include "q8_index.h"
#include <mutex>

// Block `member` of a set owns hidden units 32 member .. + 31 of one direction, for the set's sentences ("slots"), in
// groups of up to 16, one group after the other at every time step.  A time step of a group:
//   wave w polls the states that the members of the set published for slot w at the step before (one wave, so that the
//   slot's maximum needs no other wave), quantizes them and leaves the codes in LDS;
//   wave (rt, kp), rt = 2 gate + unit tile, of the first twelve multiplies its 16 weight rows by one half of the k range
//   (at most 512 bytes), the sums cross to the (slot, unit) threads through LDS;
//   eight waves apply the gates, store the new states and publish them.
// With several groups, the next group's words are requested before this one's products.  Arithmetic of
// enc_quantize_kernel, the panel product and enc_gates_kernel, value for value.
//
// What orders the accesses to LDS: two barriers per group, behind the codes and behind the products.  Codes are written in front of
// the first and read between the two, sums written between the two and read behind the second, states belong to one thread.
// Scales are written in front of the first barrier and read behind the second, where the waves without gates are on the next
// group's scales already; so two sets of them take turns (q8_enc_scale), and the next write to a set lies behind a
// barrier that every reader has passed.  (With one group the words polled are this block's own as well, whose gates come
// first; with several they are another group's, and nothing but the sets' turn orders the two.)
//
// Exchange.  A word is the float itself, or ENCG_ABSENT (a NaN pattern that is never published) while it is not there.
// Three buffers take turns.  A block that has read the words of step t - 1 knows that every member has read those of
// step t - 2 (it published t - 1 after that), so it puts its own words of that buffer back to ENCG_ABSENT, for step
// t + 1 to be published there, and waits for those stores before it publishes step t: whoever polls for step t + 1 has
// seen step t, and so no word of step t - 2.  Only the first buffer has to be clear on entry.  All of it with
// agent-scope loads and stores, so it does not matter where the blocks run; but the members of a set are block numbers
// that agree modulo 8, which are dealt to one XCD, and 1024 words exchanged by 32 blocks within an XCD arrive in 0.73 us
// where 32 blocks all over the device take 1.0 and 128 blocks 1.3.
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
// The chain of a step bounds it (1024 units, 16 slots, in us: words there 1.1, codes 0.35, products 0.45, gates 0.6), with
// several groups the instructions of the codes and the gates (2.0 us per group).  A launch per position, whose blocks read
// weights and states again, took 5.6 us at 64 sentences.  q8_encode_batch, sentences of 10 to 60 words, E = 512, us,
// launches per position -> this kernel: H = 1024, 2 / 16 / 64 / 128 / 200 / 400 sentences 244 / 354 / 411 / 595 / 880 / 1817 ->
// 127 / 171 / 241 / 393 / 681 / 1309; H = 512, 64 / 200: 390 / 580 -> 197 / 378; H = 256: 380 / 410 -> 184 / 250.
// Not kept: waves of one unit tile and a quarter of the k range that multiply all three gates (a third of the LDS reads,
// more sums to add up: 1 us faster in nothing, 5 slower where a poll comes early); all floats of a step exchanged as
// (float, tag) pairs (twice the bytes).  The pause before the first poll: too early costs another 64 KB per block and slows
// the stores that are waited for (64 sentences, 4 / 8 / 12 / 16 times 64 clocks: 263 / 242 / 240 / 242 us; 16: 196 / 173 / 173 / 180).
#define ENCG_UNITS Q8_ENC_UNITS
#define ENCG_SLOTS Q8_ENC_SLOTS
#define ENCG_THREADS 1024
#define ENCG_PITCH Q8_ENC_PITCH
#define ENCG_TILE Q8_ENC_TILE
#define ENCG_ABSENT 0xffffffffu
#define ENCG_SPINS 4096                // polls of a wait at most (some 5 ms): what follows is slow, not wrong
#define ENCG_AGENT_LOAD 0x10            // cache policy of a device-coherent load or store (sc1)

// The turn on a device (a module's variable, so one per device and process): how many of the last eight blocks (one per XCD;
// blocks of lower index start earlier) of the encoder whose turn it is have started.  Whoever takes an eight from it has the
// next turn; fewer are put back.  The wait ends after ENCG_TURN of the 100 MHz clock (an encoder that failed to launch, or
// whose blocks wait for room behind long kernels): whoever goes on then passes on an eight of its own, so nobody else
// waits for what never comes.  40 ms: an encoder whose blocks wait for room waits for another to end, and 512 sentences of
// 1024 words, the most that one launch takes, are 28 ms.
#define ENCG_TURN 4000000ull
__device__ unsigned enc_group_turn = 8;

// Clears [words, words + n) and waits for the turn.
__global__ __launch_bounds__(256) void enc_group_clear_kernel(unsigned *words, int n)
{
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
    const float *bh[2], *gx[2];          // [3H] or NULL; [L x 3H]
    const int *sent_off;                 // [S + 1]
    float *enc_h;                        // [L x 2H]
    unsigned *words;                     // [3][2][S][H], the first third ENCG_ABSENT on entry
    unsigned *ctl;                       // [sets][2]: members that left, a wait that gave up; ENCG_ABSENT on entry
    int S, H, ld, members, sets_per_dir, spin_limit, pause;
    float wh_scale[2];
};

__global__ __launch_bounds__(ENCG_THREADS) void enc_group_kernel(EncGroupArgs a)
{
    extern __shared__ __align__(16) int8_t s_codes[];                  // [16][ENCG_PITCH], sums, states, offsets, lengths
    __shared__ float s_scale[2 * ENCG_SLOTS];
    __shared__ int s_flag, s_max;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, gq = lane >> 4;
    const int H = a.H, S = a.S, ld = a.ld, members = a.members;
    const int round = (int)blockIdx.x >> 3, member = round % members, set = ((int)blockIdx.x & 7) + 8 * (round / members);
    if (blockIdx.x + 8 >= gridDim.x && tid == 0) __hip_atomic_fetch_add(&enc_group_turn, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (set >= 2 * a.sets_per_dir) return;
    // the set's slots, in groups of gs
    const int d = set & 1, c0 = S * (set >> 1) / a.sets_per_dir, ns = S * ((set >> 1) + 1) / a.sets_per_dir - c0;
    const int ng = (ns + ENCG_SLOTS - 1) / ENCG_SLOTS, gs = (ns + ng - 1) / ng;
    int *s_e = (int *)(s_codes + ENCG_SLOTS * ENCG_PITCH);
    float *s_h = (float *)(s_e + 12 * ENCG_TILE);                      // [ng][16][32] this block's states
    int *s_off = (int *)(s_h + ng * ENCG_SLOTS * ENCG_UNITS), *s_len = s_off + ng * ENCG_SLOTS;      // [ng][16]
    if (tid == 0) { s_flag = 0; s_max = 0; }
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
        const int unit0 = u0 + 16 * ut;
        const bool tiled = a.Wht[d] != nullptr && H % 16 == 0, in = wave < 12;            // (a tile of 16 rows then belongs to one gate)
        const __amdgpu_buffer_rsrc_t rw = q8_rsrc(tiled ? a.Wht[d] : a.Wh[d], (size_t)(tiled ? (3 * H + 15) / 16 * 16 : 3 * H) * ld);
        const unsigned row0 = (unsigned)(gate * H + unit0), step = tiled ? 1024u : 64u;
        const unsigned base = tiled ? ((row0 >> 4) * (unsigned)(ld >> 6) << 10) + 16u * lane : (row0 + i) * (unsigned)ld + 16u * gq;
        const bool ok = in && (tiled ? unit0 : unit0 + i) < H;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int k = kp * 8 + s;
            const unsigned off = ok && 64 * k + (tiled ? 0 : 16 * gq) < ld ? base + step * k : Q8_OOB;
            av[s] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)off, 0, 0));
        }
    };
    // one wave, iteration it (groups of time steps, counted): the codes and the scale of its slot's state, floats 4 (lane + 64 c) .. (zero past H)
    auto codes = [&](const float4 (&v)[4], int it) {
        float m = 0.0f;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(v[c].x), "v"(v[c].y));
            asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(v[c].z), "v"(v[c].w));
        }
        m = wave_max_f(m);
        float scale, inv;
        q8_scale_of(m, scale, inv);
        if (lane == 0) s_scale[q8_enc_scale(it, wave)] = scale;
#pragma unroll
        for (int c = 0; c < 4; ++c) *(int *)(s_codes + wave * ENCG_PITCH + 4 * (lane + 64 * c)) = q8_pack4(v[c].x, v[c].y, v[c].z, v[c].w, inv);
    };
    // (k steps past the rows have zero weights: whatever the codes are there, they add nothing, and no branch makes the wave
    // wait for every operand by itself)
    auto products = [&]() {
        if (wave < 12) {
            v4i acc[2] = {(v4i){0, 0, 0, 0}, (v4i){0, 0, 0, 0}};
            const int8_t *bp = s_codes + i * ENCG_PITCH + kp * 512 + 16 * gq;
#pragma unroll
            for (int s = 0; s < 8; ++s) acc[s & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[s], *(const v4i *)(bp + 64 * s), acc[s & 1], 0, 0, 0);
            // lane (i, gq) holds units 4 gq + r, r = 0..3, of slot i
            *(v4i *)(s_e + wave * ENCG_TILE + i * 16 + 4 * gq) = acc[0] + acc[1];
        }
    };
    const int sl = tid >> 5, u = tid & 31;                             // this thread's (slot, unit) pair, below 16 x 32
    auto gates = [&](const float (&gx)[3], const float (&bias)[3], float h_prev, int it) {
        const float ch = a.wh_scale[d] * s_scale[q8_enc_scale(it, sl)];
        float gh[3];
#pragma unroll
        for (int gt = 0; gt < 3; ++gt) {
            const int at = (gt * 2 + (u >> 4)) * ENCG_TILE + sl * 16 + (u & 15);
            float y = (float)(s_e[at] + s_e[at + 6 * ENCG_TILE]) * ch;
            if (a.bh[d]) y = y + bias[gt];
            gh[gt] = y;
        }
        return gru_gates(gx, gh, h_prev);
    };
    auto biases = [&](int unit, float (&bias)[3]) {
#pragma unroll
        for (int gt = 0; gt < 3; ++gt) bias[gt] = a.bh[d] && unit < H ? a.bh[d][gt * H + unit] : 0.0f;
    };
    // row of enc_h (and of gx) of step t of a slot of length l that begins at o, and the row before it
    auto row = [&](int o, int l, int t) { return d == 0 ? o + t : o + l - 1 - t; };
    const int back = d == 0 ? -1 : 1, col0 = d == 0 ? H : 0;

    // ---- all positions ----
    {
        const int unit = member * ENCG_UNITS + u;
        const bool pair = sl < ENCG_SLOTS && unit < H;
        float bias[3];
        weights(member * ENCG_UNITS);
        biases(unit, bias);
        __syncthreads();
        const int max_l = s_max;
        // words of this direction: byte offsets of the buffers of steps t - 1, t, t + 1, which take turns; all below 2^31
        const unsigned third = (unsigned)S * (unsigned)H * 8u;
        const __amdgpu_buffer_rsrc_t rx = q8_rsrc(a.words, (size_t)3 * third);
        unsigned was = 2 * third + d * (third >> 1), now = d * (third >> 1), next = third + d * (third >> 1);
        // this wave's slot of group g: its words of a step, floats 4 (lane + 64 c) .. (past H: zero, which is there)
        unsigned at[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) at[c] = 4 * (lane + 64 * c) < H ? (unsigned)((c0 + wave) * H + 4 * (lane + 64 * c)) * 4u : Q8_OOB;
        const unsigned group = (unsigned)(gs * H) * 4u;
        v4u w4[4];
        auto request = [&](unsigned buffer) {
            asm volatile("" ::: "memory");                             // (every request is made)
#pragma unroll
            for (int c = 0; c < 4; ++c) w4[c] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)at[c], (int)buffer, ENCG_AGENT_LOAD));
        };
        const unsigned mine = (unsigned)((c0 + sl) * H + unit) * 4u;
        bool gave_up = false;
        int it = 0;
        for (int t = 0; t < max_l && !gave_up; ++t) {
            for (int g = 0; g < ng; ++g, ++it) {
                const int e0 = g * ENCG_SLOTS, e = min(e0 + sl, ng * ENCG_SLOTS - 1), l = s_len[e], pos = row(s_off[e], l, t);
                const bool on = pair && t < l;
                const float *gp = a.gx[d] + (size_t)(on ? pos : 0) * 3 * H + (on ? unit : 0);
                float gx[3];
#pragma unroll
                for (int gt = 0; gt < 3; ++gt) gx[gt] = gp[gt * H];
                if (t < s_len[e0 + wave]) {                            // wave-uniform
                    float4 v[4];
                    bool there = true;
                    if (t > 0) {
                        if (ng == 1) {
                            if (a.spin_limit > 1)
                                for (int p = 0; p < a.pause; ++p) __builtin_amdgcn_s_sleep(1);
                            request(was);
                        }
                        for (int spins = 1;; ++spins) {
                            unsigned m = 0;                            // (an absent word is the largest there is)
#pragma unroll
                            for (int c = 0; c < 4; ++c) m = max(max(m, max(w4[c].x, w4[c].y)), max(w4[c].z, w4[c].w));
                            if (!__any(m == ENCG_ABSENT)) break;
                            if (spins >= a.spin_limit ||
                                ((spins & 63) == 0 && __hip_atomic_load(a.ctl + 2 * set + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != ENCG_ABSENT)) {
                                if (lane == 0) {
                                    s_flag = 1;
                                    __hip_atomic_store(a.ctl + 2 * set + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                }
                                there = false;
                                break;
                            }
                            request(was + g * group);
                        }
#pragma unroll
                        for (int c = 0; c < 4; ++c) v[c] = __builtin_bit_cast(float4, w4[c]);
                    } else {
#pragma unroll
                        for (int c = 0; c < 4; ++c) v[c] = make_float4(0.f, 0.f, 0.f, 0.f);
                    }
                    if (there) codes(v, it);
                }
                __syncthreads();
                if (s_flag) { gave_up = true; break; }
                if (on && t + 2 < l) __builtin_amdgcn_raw_buffer_store_b32(ENCG_ABSENT, rx, (int)(mine + g * group), (int)next, ENCG_AGENT_LOAD);
                if (ng > 1) {                                          // the next group's words, under this one's products and gates
                    const bool wrap = g + 1 == ng;
                    if (t + wrap > 0 && t + wrap < s_len[wrap ? wave : e0 + ENCG_SLOTS + wave]) request(wrap ? now : was + (g + 1) * group);
                }
                products();
                __syncthreads();
                if (tid < ENCG_SLOTS * ENCG_UNITS) {
                    const float hn = gates(gx, bias, s_h[e0 * ENCG_UNITS + tid], it);
                    if (on) {
                        unsigned word = __float_as_uint(hn);
                        word = word == ENCG_ABSENT ? 0x7fffffffu : word;
                        q8_stores_performed();
                        if (t + 1 < l) __builtin_amdgcn_raw_buffer_store_b32(word, rx, (int)(mine + g * group), (int)now, ENCG_AGENT_LOAD);
                        a.enc_h[(size_t)pos * 2 * H + col0 + unit] = hn;
                        s_h[e0 * ENCG_UNITS + tid] = hn;
                    }
                }
            }
            const unsigned first = was;
            was = now;
            now = next;
            next = first;
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
            const int e0 = g * ENCG_SLOTS, lw = s_len[e0 + wave];
            if (t < lw) {
                const float *h = a.enc_h + (size_t)(row(s_off[e0 + wave], lw, t) + back) * 2 * H + col0;
                float4 v[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int k = 4 * (lane + 64 * c);
                    v[c] = t > 0 && k < H ? *(const float4 *)(h + k) : make_float4(0.f, 0.f, 0.f, 0.f);
                }
                codes(v, 0);
            }
            for (int m = 0; m < members; ++m) {
                const int unit = m * ENCG_UNITS + u, at = min(e0 + sl, ng * ENCG_SLOTS - 1), l = s_len[at], pos = row(s_off[at], l, t);
                weights(m * ENCG_UNITS);
                __syncthreads();
                products();
                __syncthreads();
                if (sl < ENCG_SLOTS && unit < H && t < l) {
                    float bias[3];
                    biases(unit, bias);
                    const float *gp = a.gx[d] + (size_t)pos * 3 * H + unit;
                    const float gx[3] = {gp[0], gp[H], gp[2 * H]};
                    a.enc_h[(size_t)pos * 2 * H + col0 + unit] = gates(gx, bias, t > 0 ? a.enc_h[(size_t)(pos + back) * 2 * H + col0 + unit] : 0.0f, 0);
                }
            }
            __syncthreads();
        }
}

// =================================================================== host launchers ==

// 4-byte words of scratch (0: not for this shape): the members' words and the sets' counters and flags.
size_t q8i_enc_group_words(const q8_gru_weights *fwd, const q8_gru_weights *bwd, int S, int max_l)
{
    const int H = fwd->Wh.cols;
    int members, sets, groups, slots;
    if (H % 4 || H > 1024 || fwd->Wh.ld > 1024 || bwd->Wh.ld != fwd->Wh.ld || !q8_enc_one_launch(H, S, max_l)) return 0;
    q8_enc_plan(H, S, &members, &sets, &groups, &slots);
    return (size_t)6 * S * H + 4 * sets;
}

q8_status q8i_enc_group(q8_ctx *ctx, const q8_gru_weights *fwd, const q8_gru_weights *bwd, const int *sent_off, int S, float *enc_h,
                        const float *gxf, const float *gxb, unsigned *words)
{
    const int H = fwd->Wh.cols;
    int members, spd, ng, gs;
    const size_t lds = q8_enc_plan(H, S, &members, &spd, &ng, &gs);
    const int clear = 4 * spd + 2 * S * H;
    // (the two launches side by side on their queue: a stream that shares it cannot wait for the turn between them)
    static std::mutex pair;
    std::lock_guard<std::mutex> hold(pair);
    hipLaunchKernelGGL(enc_group_clear_kernel, dim3(1 + (clear + 255) / 256), dim3(256), 0, ctx->stream, words, clear);
    const q8_status st = q8i_launch_check(ctx, "clear");
    if (st) return st;
    EncGroupArgs a = {{fwd->Wh.data, bwd->Wh.data}, {fwd->Wh.tiles, bwd->Wh.tiles}, {fwd->bh, bwd->bh}, {gxf, gxb}, sent_off, enc_h,
                      words + 4 * spd, words, S, H, fwd->Wh.ld, members, spd, ctx->enc_spin_limit < ENCG_SPINS ? ctx->enc_spin_limit : ENCG_SPINS,
                      (size_t)gs * H > 8192 ? 11 : 8, {fwd->Wh.scale, bwd->Wh.scale}};
    Q8_LAUNCH(ctx, Q8_KERNEL_GRU, enc_group_kernel, dim3(8 * members * ((2 * spd + 7) / 8)), dim3(ENCG_THREADS), lds, a);
    return q8i_launch_check(ctx, "encoder recurrences");
}
