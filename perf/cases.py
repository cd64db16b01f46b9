"""What this library is timed on: the calls a program makes that lets games be played, observed, stored and scored on one GPU.

Every case goes through the public entry points.  A pass of the playing paths advances the same games further, so every
pass works on states that no pass has seen before; the seed fixes the walls and the random policy, hence every output.
All results are whole numbers, or whole numbers times 0.001f, so they are compared exactly.
"""
import math

import torch

import paper_2605_20577_amd as mj
from paper_2605_20577_amd import binding

RECORD = mj.ENV_DTYPE.itemsize                    # canonical record of one game
TOKENS = 4 * mj.TOKEN_DTYPE.itemsize              # token observation of one game, four viewers
PLANES = 4 * 56 * 34                              # plane observation of one game, four viewers
QUERY, RESULT = mj.QUERY_DTYPE.itemsize, mj.RESULT_DTYPE.itemsize
EXTRA = mj.F_ENDGAME | mj.F_KANDORA_LATE | mj.F_NAGASHI | mj.F_ANKAN_ROB | mj.F_PAO
RULES = {"nored": mj.RULES_NORED, "red": mj.RULES_RED, "red+": mj.RULES_RED | EXTRA}
MODES = {"single": mj.MODE_SINGLE, "east": mj.MODE_EAST, "half": mj.MODE_HALF}
SETTLE = 1024                                     # untimed steps, longer than a hanchan, so that games are spread over all rounds


def listed():
    return [
        # A debugging or unit-test sized run: 256 single rounds, everything decided by launches and the chain of one step.
        {"name": "rollout_256_single", "path": "rollout", "games": 256, "rules": "nored", "mode": "single", "steps": 128},
        # The headline workload: a long random-policy run of 65,536 whole games, then the records of all of them.
        {"name": "rollout_65536_nored", "path": "rollout", "games": 65536, "rules": "nored", "mode": "half", "steps": 2048},
        # The same with red fives and abortive draws, at a length a data generator would ask for between two reads.
        {"name": "rollout_65536_red", "path": "rollout", "games": 65536, "rules": "red", "mode": "half", "steps": 512},
        # A caller that advances a large pool by a few random moves and then looks at masks, rewards and standings.
        {"name": "advance_65536_20", "path": "advance", "games": 65536, "rules": "nored", "mode": "half", "steps": 20},
        # The same with every rule flag on and a batch that fills neither blocks nor the machine evenly.
        {"name": "advance_110001_flags", "path": "advance", "games": 110001, "rules": "red+", "mode": "half", "steps": 50},
        # Whole-game evaluation of agents, 1,000 games at a time: masks, planes, step, rewards, standings, restarts.
        {"name": "arena_1000", "path": "arena", "games": 1000, "rules": "red", "mode": "east", "steps": 1},
        # An agent's training loop with the token observation, one launch per library call and step.
        {"name": "tokens_65536", "path": "tokens", "games": 65536, "rules": "red", "mode": "half", "steps": 1},
        # The largest batch, the plane observation written after every step.
        {"name": "planes_1048576", "path": "planes", "games": 1 << 20, "rules": "red", "mode": "half", "steps": 4},
        # A checkpoint: every game written to records, the records read into a second batch that goes on from there.
        {"name": "checkpoint_65536", "path": "checkpoint", "games": 65536, "rules": "red", "mode": "half", "steps": 1},
        # A server that scores a few hands per request, without a handle.
        {"name": "hands_1000", "path": "hands_static", "hands": 1000},
        # A large batch of hands, half random draws, half complete.
        {"name": "hands_1048576", "path": "hands", "hands": 1 << 20},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["rollout", "rollout", "advance", "advance", "arena", "tokens", "planes", "checkpoint", "hands", "hands_static"])
    if path == "hands":
        return {"path": path, "hands": _log(rng, 1, 1 << 20)}
    if path == "hands_static":
        return {"path": path, "hands": _log(rng, 1, 1 << 17)}
    case = {"path": path, "rules": rng.choice(["nored", "red", "red+"]), "mode": rng.choice(["single", "east", "half", "half"]), "steps": 1}
    if path == "rollout":
        case["games"] = _log(rng, 64, 200000)
        case["steps"] = _log(rng, 128, min(2048, 65536 * 2048 // case["games"]))
    elif path == "advance":
        case["games"] = _log(rng, 64, 1 << 18)
        case["steps"] = _log(rng, 1, 100)
    elif path == "arena":
        case["games"] = _log(rng, 1, 20000)
    elif path == "tokens":
        case["games"] = _log(rng, 64, 1 << 18)
    elif path == "planes":
        case["games"] = _log(rng, 1000, 1 << 19)
        case["steps"] = rng.randint(1, 8)
    else:
        case["games"] = _log(rng, 64, 1 << 17)
    return case


def _hands(n, seed):
    """n query records on the GPU: the first half 14 tiles drawn from a full wall, the second half complete hands of four sets
    (up to three of them exposed) and a pair, with random winds, situation and dora indicators"""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def ints(lo, hi, *shape):
        return torch.randint(lo, hi, shape, generator=gen, device=dev)

    def below(p):
        return torch.rand(n, generator=gen, device=dev) < p

    q = torch.zeros((n, QUERY), dtype=torch.uint8, device=dev)
    field = {name: mj.QUERY_DTYPE.fields[name][1] for name in mj.QUERY_DTYPE.names}

    def put(name, value, lo=0):
        v = value.reshape(value.shape[0], -1).to(torch.uint8)
        q[lo:lo + v.shape[0], field[name]:field[name] + v.shape[1]] = v

    half = n // 2
    if half:
        kinds = torch.rand((half, 136), generator=gen, device=dev).topk(14, dim=1).indices >> 2
        put("hand", torch.zeros((half, 34), dtype=torch.int64, device=dev).scatter_add_(1, kinds, torch.ones_like(kinds)))
        put("win_kind", kinds[:, 0])
    need, parts = n - half, []
    while need > 0:
        m = need + need // 2 + 64
        hand = torch.zeros((m, 34), dtype=torch.int64, device=dev)
        total, one = torch.zeros_like(hand), torch.ones((m, 1), dtype=torch.int64, device=dev)
        melds = torch.zeros((m, 4), dtype=torch.int64, device=dev)
        n_meld = ints(0, 4, m)
        for j in range(4):
            run, exposed = ints(0, 2, m).bool(), j < n_meld
            kind = torch.where(run, 9 * ints(0, 3, m) + ints(0, 7, m), ints(0, 34, m))
            for d in range(3):
                at = (kind + torch.where(run, d, 0)).unsqueeze(1)
                total.scatter_add_(1, at, one)
                hand.scatter_add_(1, at, (~exposed).long().unsqueeze(1))
            form = torch.where(run, torch.ones_like(kind), torch.tensor([2, 4, 3], device=dev)[ints(0, 3, m)])
            total.scatter_add_(1, kind.unsqueeze(1), (exposed & (form >= 3)).long().unsqueeze(1))
            word = form | kind << 3 | ints(1, 4, m) << 9 | torch.where(run, ints(0, 3, m), 0) << 11
            melds[:, j] = torch.where(exposed, word, 0)
        pair = ints(0, 34, m).unsqueeze(1)
        total.scatter_add_(1, pair, 2 * one)
        hand.scatter_add_(1, pair, 2 * one)
        win = (torch.rand((m, 34), generator=gen, device=dev) * hand).argmax(dim=1)
        ok = torch.nonzero(total.amax(dim=1) <= 4).flatten()[:need]
        parts.append((hand[ok], melds[ok], n_meld[ok], win[ok]))
        need -= ok.numel()
    hand, melds, n_meld, win = (torch.cat(p) for p in zip(*parts))
    put("hand", hand, half)
    put("meld", torch.stack((melds & 255, melds >> 8), dim=2), half)
    put("n_meld", n_meld, half)
    put("win_kind", win, half)
    flags = below(0.5).long()
    for bit, p in ((1, 0.3), (2, 0.05), (3, 0.05), (4, 0.05), (5, 0.05), (6, 0.02)):
        flags |= below(p).long() << bit
    put("flags", flags)
    put("riichi", ints(1, 3, n) * below(0.5))
    put("seat_wind", ints(0, 4, n))
    put("round_wind", ints(0, 2, n))
    put("n_ind", ints(1, 5, n))
    put("ind", ints(0, 34, n, 5))
    put("ura", ints(0, 34, n, 5))
    put("n_aka", ints(1, 3, n) * below(0.3))
    put("kuitan", torch.ones(n, device=dev))
    return q.reshape(-1)


def prepare(case, seed):
    path, dev = case["path"], torch.device("cuda:0")
    if path in ("hands", "hands_static"):
        state = {"path": path, "n": case["hands"], "queries": _hands(case["hands"], seed),
                 "results": torch.empty(case["hands"] * RESULT, dtype=torch.uint8, device=dev)}
        state["env"] = mj.MahjongEnv(64, seed=seed, flags=mj.RULES_RED, mode=mj.MODE_HALF)     # its tables are what is used
        return state
    B = case["games"]
    env = mj.MahjongEnv(B, seed=seed, flags=RULES[case["rules"]], mode=MODES[case["mode"]])
    env.step_random(SETTLE)
    state = {"path": path, "env": env, "steps": case["steps"]}
    if path in ("rollout", "checkpoint"):
        state["records"] = torch.empty((B, RECORD), dtype=torch.uint8, device=dev)
    if path == "checkpoint":
        state["resumed"] = mj.MahjongEnv(B, seed=seed, flags=RULES[case["rules"]], mode=MODES[case["mode"]])
    if path in ("tokens", "arena"):
        state["actions"] = torch.empty((B, 4), dtype=torch.int8, device=dev)
    if path == "tokens":
        state["tokens"] = torch.empty((B, TOKENS), dtype=torch.uint8, device=dev)
        state["out"] = (torch.empty((B, 4, 2), dtype=torch.int64, device=dev), torch.empty((B, 4), dtype=torch.int32, device=dev),
                        torch.empty((B, 4), dtype=torch.float32, device=dev), torch.empty((B,), dtype=torch.uint8, device=dev))
    if path == "planes":
        state["planes"] = torch.empty((B, 4, 56, 34), dtype=torch.uint8, device=dev)
    return state


def run(state):
    path, env = state["path"], state["env"]
    if path == "rollout":
        env.step_random(state["steps"])
        binding.mj_export(env._h, 0, env.B, state["records"])
        return state["records"]
    if path == "advance":
        env.step_random(state["steps"])
        return env.legal_mask(), env.reward(), env.standings()
    if path == "arena":
        mask, planes = env.legal_mask(), env.observe()
        env.sample_random(state["actions"])
        env.step(state["actions"])
        reward, standings = env.reward(), env.standings()
        env.reset_done()
        return mask, planes, state["actions"], reward, standings
    if path == "tokens":
        env.sample_random(state["actions"])
        env.step_full(state["actions"], True, state["out"])
        env.observe_tokens(state["tokens"])
        return state["actions"], state["out"], state["tokens"]
    if path == "planes":
        env.step_random(state["steps"], True, state["planes"])
        return state["planes"], env.reward()
    if path == "checkpoint":
        binding.mj_export(env._h, 0, env.B, state["records"])
        binding.mj_import(state["resumed"]._h, 0, env.B, state["records"])
        return state["records"], state["resumed"].legal_mask(), state["resumed"].standings()
    if path == "hands":
        env.eval_hands_device(state["queries"], state["results"])
    else:
        binding.mj_eval_hands_static(state["n"], state["queries"], state["results"])
    return state["results"]


def work(case):
    """bytes: inputs read once, outputs written once; a game's state counts as its record.  There is no floating-point work:
    the games are whole-number logic, which this figure does not price."""
    path = case["path"]
    if path in ("hands", "hands_static"):
        return {"bytes": case["hands"] * (QUERY + RESULT), "flops": 0}
    B = case["games"]
    masks, reward, standings, actions = 64, 33, 20, 4
    per_game = {"rollout": 3 * RECORD, "advance": 2 * RECORD + masks + reward + standings,
                "arena": 2 * RECORD + masks + PLANES + 2 * actions + reward + standings,
                "tokens": 2 * RECORD + 2 * actions + masks + reward + TOKENS,
                "planes": 2 * RECORD + case["steps"] * PLANES + reward,
                "checkpoint": 4 * RECORD + masks + standings}[path]
    return {"bytes": B * per_game, "flops": 0}


def tolerance(case):
    return "exact"
