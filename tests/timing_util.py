"""Comparisons of times: a fault shows in every attempt, a disturbance from outside in one."""


def below(compare, attempts=4):
    """compare() returns a time and what it has to stay below; whether it does in one of a few attempts."""
    for _ in range(attempts):
        took, limit = compare()
        print(f"{took:.4g}, to stay below {limit:.4g}", flush=True)
        if took < limit:
            return True
    return False
